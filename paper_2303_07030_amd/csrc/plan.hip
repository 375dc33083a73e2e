// Work plans for the segmented reductions (built once per sparsity pattern).
//
// A plan cuts the entries of a sorted sparse operand (the rows of a CSR or
// the columns of a CSC) into work items of about L entries:
//   * a short segment (1 <= length <= S = L + min(L, 32)) is never split;
//     consecutive short segments are packed into one item while their merged
//     cost (entries + one per segment) starts inside the same window of L;
//   * a long segment (length > S) is cut into chunks of L entries, one item
//     each, whose partial sums are combined afterwards in chunk order;
//   * empty segments get no item; they are listed for a zero fill.
// Work per item is therefore bounded by L + S entries whatever the length
// distribution, and only long segments ever need a second pass.
//
// Construction (all on the GPU):
//   cost_r  = length + 1 for a short segment, L for a long one, 0 if empty;
//   pos_r   = exclusive sum of cost; window g_r = pos_r / L;
//   a short segment starts an item unless the nonempty segment before it is
//   short and lies in the same window; the L added for a long segment always
//   moves the next short segment to a new window, so no item spans a long
//   segment;
//   items per segment: ceil(length / L) if long, 1 if it starts a group;
//   exclusive sums give every item's index and entry offset, and list the
//   long segments, the huge ones (more than kHugeChunks chunks, combined by a
//   whole block instead of one wave), every chunk item and the empty
//   segments.
// Three launches over the segment pointers: the blocks' cost totals; from
// their prefix, the blocks' item and list totals; from both prefixes, the
// plan itself.  Each block takes one contiguous range of segments and
// recomputes what it needs from the pointers (L2 resident), so nothing per
// segment is stored in between.
#include <algorithm>

#include "nsd_internal.hpp"

namespace nsd {

constexpr int kPlanThreads = 256;
constexpr int kHugeChunks = 64;

// A segment is long (chunked) above L + min(L, 32) entries: keeping slightly
// longer segments whole spares the combine pass to most moderate lengths at
// small L, while items stay near L entries at large L (measured on MI355X).
__host__ __device__ __forceinline__ int64_t short_max(int32_t L) {
    return (int64_t)L + (L < 32 ? L : 32);
}
__device__ __forceinline__ bool seg_long(int32_t len, int32_t L) { return len > short_max(L); }

constexpr int kPlanWaves = kPlanThreads / kWave;
constexpr int kPlanPer = 4;                             // segments per thread and step
constexpr int kPlanStep = kPlanThreads * kPlanPer;
constexpr int kPlanMaxBlocks = 1024;
// Chunks that a long segment's own thread writes; more are written by a wave.
constexpr int kPlanOwnChunks = 8;

// Segments of one block (a multiple of a step).
static int64_t plan_per_block(int64_t nseg) {
    return ceil_div(ceil_div(nseg, kPlanMaxBlocks), kPlanStep) * kPlanStep;
}

// What is summed over segments before one (cost, last nonempty segment by
// maximum), and what is counted from it.
constexpr int kPlanCounts = 5;  // items, long, empty, chunk items, huge
struct PlanCost {
    int32_t cost, last;
};
struct PlanCounts {
    int32_t n[kPlanCounts];
};

// Inclusive scans over a wave.
__device__ __forceinline__ int32_t plan_wave_sum(int32_t x, int lane) {
#pragma unroll
    for (int d = 1; d < kWave; d <<= 1) {
        const int32_t y = __shfl_up(x, d, kWave);
        if (lane >= d) x += y;
    }
    return x;
}
__device__ __forceinline__ int32_t plan_wave_max(int32_t x, int lane) {
#pragma unroll
    for (int d = 1; d < kWave; d <<= 1) {
        const int32_t y = __shfl_up(x, d, kWave);
        if (lane >= d) x = max(x, y);
    }
    return x;
}

// Maximum over the block (nonnegative values).
__device__ __forceinline__ int32_t plan_block_max(int32_t x) {
    __shared__ int32_t w[kPlanWaves];
    const int lane = threadIdx.x & (kWave - 1);
    x = plan_wave_max(x, lane);
    if (lane == kWave - 1) w[threadIdx.x / kWave] = x;
    __syncthreads();
    x = 0;
    for (int i = 0; i < kPlanWaves; ++i) x = max(x, w[i]);
    __syncthreads();
    return x;
}

// Exclusive scan over the block of one PlanCost per thread; tot: the block's.
__device__ __forceinline__ PlanCost plan_scan_cost(PlanCost v, PlanCost &tot) {
    __shared__ PlanCost w[kPlanWaves];
    const int lane = threadIdx.x & (kWave - 1), wave = threadIdx.x / kWave;
    const int32_t c = plan_wave_sum(v.cost, lane), l = plan_wave_max(v.last, lane);
    if (lane == kWave - 1) w[wave] = {c, l};
    __syncthreads();
    PlanCost pre{0, -1};
    tot = {0, -1};
    for (int i = 0; i < kPlanWaves; ++i) {
        if (i < wave) pre = {pre.cost + w[i].cost, max(pre.last, w[i].last)};
        tot = {tot.cost + w[i].cost, max(tot.last, w[i].last)};
    }
    const int32_t up = __shfl_up(l, 1, kWave);
    __syncthreads();
    return {pre.cost + c - v.cost, lane > 0 ? max(pre.last, up) : pre.last};
}

// Exclusive scan over the block of one PlanCounts per thread.
__device__ __forceinline__ PlanCounts plan_scan_counts(PlanCounts v, PlanCounts &tot) {
    __shared__ PlanCounts w[kPlanWaves];
    const int lane = threadIdx.x & (kWave - 1), wave = threadIdx.x / kWave;
    PlanCounts inc;
#pragma unroll
    for (int j = 0; j < kPlanCounts; ++j) inc.n[j] = plan_wave_sum(v.n[j], lane);
    if (lane == kWave - 1) w[wave] = inc;
    __syncthreads();
    PlanCounts out;
#pragma unroll
    for (int j = 0; j < kPlanCounts; ++j) {
        int32_t pre = 0, all = 0;
        for (int i = 0; i < kPlanWaves; ++i) {
            if (i < wave) pre += w[i].n[j];
            all += w[i].n[j];
        }
        out.n[j] = pre + inc.n[j] - v.n[j];
        tot.n[j] = all;
    }
    __syncthreads();
    return out;
}

// This thread's segments of a step: kPlanPer consecutive ones from r0.
struct PlanSegs {
    int32_t beg[kPlanPer], len[kPlanPer], cost[kPlanPer];
    PlanCost sum;
    __device__ __forceinline__ PlanSegs(const int32_t *segptr, int64_t r0, int64_t end, int32_t L) {
        int32_t p[kPlanPer + 1];
#pragma unroll
        for (int u = 0; u <= kPlanPer; ++u) p[u] = segptr[min(r0 + u, end)];
        sum = {0, -1};
#pragma unroll
        for (int u = 0; u < kPlanPer; ++u) {
            beg[u] = p[u];
            len[u] = p[u + 1] - p[u];  // 0 past the end
            cost[u] = len[u] == 0 ? 0 : (seg_long(len[u], L) ? L : len[u] + 1);
            sum.cost += cost[u];
            if (len[u] > 0) sum.last = (int32_t)(r0 + u);
        }
    }
};

__global__ __launch_bounds__(kPlanThreads) void plan_cost_kernel(int32_t nseg, int64_t per,
                                                                 const int32_t *segptr, int32_t L,
                                                                 PlanCost *sums) {
    const int64_t b0 = (int64_t)blockIdx.x * per, b1 = min(b0 + per, (int64_t)nseg);
    PlanCost s{0, -1};
    for (int64_t r = b0 + (int64_t)threadIdx.x * kPlanPer; r < b1; r += kPlanStep) {
        const PlanSegs g(segptr, r, b1, L);
        s = {s.cost + g.sum.cost, max(s.last, g.sum.last)};
    }
    PlanCost tot;
    plan_scan_cost(s, tot);
    if (threadIdx.x == 0) sums[blockIdx.x] = tot;
}

// The cost and last nonempty segment before this block.
__device__ __forceinline__ PlanCost plan_cost_before(const PlanCost *sums) {
    PlanCost s{0, -1}, tot;
    for (int j = threadIdx.x; j < (int)blockIdx.x; j += kPlanThreads)
        s = {s.cost + sums[j].cost, max(s.last, sums[j].last)};
    plan_scan_cost(s, tot);
    return tot;
}

// The counts of this thread's segments, given the cost and the last nonempty
// segment before its first one.
__device__ __forceinline__ PlanCounts plan_count(const PlanSegs &g, const int32_t *segptr, int32_t L,
                                                 int64_t r0, int64_t end, PlanCost at,
                                                 int32_t (&items)[kPlanPer], int32_t &longest) {
    PlanCounts c{};
    int32_t pos = at.cost, prev = at.last;
    int32_t plen = prev >= 0 ? segptr[prev + 1] - segptr[prev] : 0;
#pragma unroll
    for (int u = 0; u < kPlanPer; ++u) {
        const int32_t len = g.len[u];
        const bool lg = seg_long(len, L);
        items[u] = 0;
        if (lg) {
            items[u] = (len + L - 1) / L;
            longest = max(longest, items[u]);
        } else if (len > 0) {
            const bool joins = prev >= 0 && !seg_long(plen, L) && (pos - plen - 1) / L == pos / L;
            items[u] = joins ? 0 : 1;
        }
        c.n[0] += items[u];
        c.n[1] += lg;
        c.n[2] += len == 0 && r0 + u < end;
        c.n[3] += lg ? items[u] : 0;
        c.n[4] += lg && items[u] > kHugeChunks;
        pos += g.cost[u];
        if (len > 0) {
            prev = (int32_t)(r0 + u);
            plen = len;
        }
    }
    return c;
}

__global__ __launch_bounds__(kPlanThreads) void plan_count_kernel(int32_t nseg, int64_t per,
                                                                  const int32_t *segptr, int32_t L,
                                                                  const PlanCost *costs,
                                                                  PlanCounts *counts,
                                                                  int32_t *longest) {
    const int64_t b0 = (int64_t)blockIdx.x * per, b1 = min(b0 + per, (int64_t)nseg);
    PlanCost run = plan_cost_before(costs), tot;
    PlanCounts sum{};
    int32_t most = 0, items[kPlanPer];
    for (int64_t s = b0; s < b1; s += kPlanStep) {
        const int64_t r0 = s + (int64_t)threadIdx.x * kPlanPer;
        const PlanSegs g(segptr, r0, b1, L);
        const PlanCost e = plan_scan_cost(g.sum, tot);
        const PlanCounts c = plan_count(g, segptr, L, r0, b1,
                                        {run.cost + e.cost, max(run.last, e.last)}, items, most);
#pragma unroll
        for (int j = 0; j < kPlanCounts; ++j) sum.n[j] += c.n[j];
        run = {run.cost + tot.cost, max(run.last, tot.last)};
    }
    PlanCounts all;
    plan_scan_counts(sum, all);
    if (threadIdx.x == 0) counts[blockIdx.x] = all;
    most = plan_block_max(most);
    if (threadIdx.x == 0) longest[blockIdx.x] = most;
}

struct PlanOut {
    int32_t *item_ptr, *long_seg, *long_first, *huge_idx, *chunk_item, *chunk_ord, *empty_seg;
};

// Items first .. first + n - 1 of a long segment at entry beg, from chunk c0
// in steps.
__device__ __forceinline__ void plan_chunks(const PlanOut &o, int32_t L, int32_t beg, int32_t first,
                                            int32_t n, int32_t cpos, int32_t c0, int32_t step) {
    for (int32_t c = c0; c < n; c += step) {
        o.item_ptr[first + c] = beg + c * L;
        o.chunk_item[cpos + c] = first + c;
        o.chunk_ord[first + c] = cpos + c;
    }
}

__global__ __launch_bounds__(kPlanThreads) void plan_fill_kernel(int32_t nseg, int32_t nnz,
                                                                 int64_t per, const int32_t *segptr,
                                                                 int32_t L, const PlanCost *costs,
                                                                 const PlanCounts *counts,
                                                                 const int32_t *longest, PlanOut o,
                                                                 int32_t *totals) {
    __shared__ int4 many[kPlanStep];  // long segments of many chunks: begin, first, n, cpos
    __shared__ int nmany;
    const int64_t b0 = (int64_t)blockIdx.x * per, b1 = min(b0 + per, (int64_t)nseg);
    PlanCost run = plan_cost_before(costs), tot;
    PlanCounts base{}, all;
    for (int j = threadIdx.x; j < (int)blockIdx.x; j += kPlanThreads)
#pragma unroll
        for (int i = 0; i < kPlanCounts; ++i) base.n[i] += counts[j].n[i];
    plan_scan_counts(base, all);
    base = all;
    for (int64_t s = b0; s < b1; s += kPlanStep) {
        const int64_t r0 = s + (int64_t)threadIdx.x * kPlanPer;
        const PlanSegs g(segptr, r0, b1, L);
        const PlanCost e = plan_scan_cost(g.sum, tot);
        int32_t items[kPlanPer], most = 0;
        const PlanCounts c = plan_count(g, segptr, L, r0, b1,
                                        {run.cost + e.cost, max(run.last, e.last)}, items, most);
        if (threadIdx.x == 0) nmany = 0;
        PlanCounts x = plan_scan_counts(c, all);  // its barriers publish nmany
#pragma unroll
        for (int i = 0; i < kPlanCounts; ++i) x.n[i] += base.n[i];
#pragma unroll
        for (int u = 0; u < kPlanPer; ++u) {
            const int64_t r = r0 + u;
            if (r >= b1) break;
            const int32_t len = g.len[u], n = items[u], first = x.n[0];
            if (seg_long(len, L)) {
                o.long_seg[x.n[1]] = (int32_t)r;
                o.long_first[x.n[1]] = first;
                if (n > kHugeChunks) o.huge_idx[x.n[4]++] = x.n[1];
                ++x.n[1];
                if (n <= kPlanOwnChunks) plan_chunks(o, L, g.beg[u], first, n, x.n[3], 0, 1);
                else many[atomicAdd(&nmany, 1)] = make_int4(g.beg[u], first, n, x.n[3]);
                x.n[3] += n;
            } else if (len > 0) {
                if (n) {
                    o.item_ptr[first] = g.beg[u];
                    o.chunk_ord[first] = -1;
                }
            } else {
                o.empty_seg[x.n[2]++] = (int32_t)r;
            }
            x.n[0] += n;
            if (r == nseg - 1) o.item_ptr[x.n[0]] = nnz;
        }
        __syncthreads();
        for (int i = threadIdx.x / kWave; i < nmany; i += kPlanWaves)
            plan_chunks(o, L, many[i].x, many[i].y, many[i].z, many[i].w,
                        threadIdx.x & (kWave - 1), kWave);
        __syncthreads();
        run = {run.cost + tot.cost, max(run.last, tot.last)};
#pragma unroll
        for (int i = 0; i < kPlanCounts; ++i) base.n[i] += all.n[i];
    }
    if (blockIdx.x == gridDim.x - 1) {  // the blocks' longest: an atomic of each took 45 us
        int32_t most = 0;
        for (int j = threadIdx.x; j < (int)gridDim.x; j += kPlanThreads) most = max(most, longest[j]);
        most = plan_block_max(most);
        if (threadIdx.x == 0) {
#pragma unroll
            for (int i = 0; i < kPlanCounts; ++i) totals[i] = base.n[i];
            totals[kPlanCounts] = most;
        }
    }
}

__global__ void plan_sentinel_kernel(int32_t *item_ptr, int32_t nnz) { item_ptr[0] = nnz; }

static size_t plan_ws_bytes() {
    Carver c(nullptr);
    c.take<PlanCost>(kPlanMaxBlocks);
    c.take<PlanCounts>(kPlanMaxBlocks);
    c.take<int32_t>(kPlanMaxBlocks);
    c.take<int32_t>(64);
    return c.bytes();
}

}  // namespace nsd

using namespace nsd;

extern "C" {

nsd_status nsd_plan_item_len(int32_t nnz, int32_t k, int32_t *item_len) {
    NSD_REQUIRE(item_len != nullptr, "item_len is NULL");
    NSD_REQUIRE(nnz >= 0 && k >= 1, "need nnz >= 0 and k >= 1");
    // about 32 waves of items per SIMD (256 CUs x 4 SIMDs), an item being
    // one slot of a wave (a slot covers min(k, 256) columns); measured on
    // MI355X this is within 2% of the best length for every workload shape
    // tried (1M to 60M entries, k = 32 to 256)
    const WidthPlan wp = narrow_plan(k, k % 4 == 0, scalar_width(nnz, k));
    const int64_t slots = 32768LL * (kWave / wp.g);
    int32_t L = 16;
    while (L < 256 && (int64_t)L * 2 * slots <= nnz) L <<= 1;
    // small inputs: if 16-entry items would not give every SIMD one wave of
    // items, shorten them (down to 2) so that the serial walk of each slot,
    // not the idle chip, sets the time (an SpMM of 10K entries at k = 16: 8.2 us
    // at L = 2 against 13.4 at L = 16)
    const int64_t fill = 1024LL * (kWave / wp.g);
    if ((int64_t)16 * fill > nnz) {
        L = 2;
        while (L < 16 && (int64_t)L * 2 * fill <= nnz) L <<= 1;
    }
    // the narrow slots of widths that are no multiple of four: longer items
    // spread a wave's metadata reads over more lines (30M entries, k = 50, us: a
    // bilinear step 1738 at 32 against 1893 at 128, the factorisation 2807 / 2936)
    if (wp.ragged && wp.g <= 16) L = std::min(L, 16 + wp.g);
    *item_len = L;
    return NSD_OK;
}

nsd_status nsd_plan_bounds(int32_t nseg, int32_t nnz, int32_t item_len, int32_t *max_items,
                           int32_t *max_long, int32_t *max_chunks, size_t *ws_bytes) {
    NSD_REQUIRE(nseg >= 0 && nnz >= 0 && item_len >= 1, "need nseg, nnz >= 0, item_len >= 1");
    NSD_REQUIRE(max_items && max_long && max_chunks && ws_bytes, "null pointer");
    if (2LL * nnz + nseg >= (1LL << 31)) return fail(NSD_ERR_TOO_LARGE, "plan cost overflows int32");
    *max_items = std::min(nseg, nnz) + 2 * (nnz / item_len) + 1;
    *max_long = nnz / (item_len + 1) + 1;
    *max_chunks = 2 * (nnz / item_len) + 1;
    *ws_bytes = plan_ws_bytes();
    return NSD_OK;
}

nsd_status nsd_plan_build(int32_t nseg, int32_t nnz, const int32_t *segptr, int32_t item_len,
                          int32_t *item_ptr, int32_t *long_seg, int32_t *long_first,
                          int32_t *huge_idx, int32_t *chunk_item, int32_t *chunk_ord,
                          int32_t *empty_seg, nsd_plan *plan, void *ws, size_t ws_bytes,
                          void *stream) {
    NSD_REQUIRE(nseg >= 0 && nnz >= 0 && item_len >= 1, "need nseg, nnz >= 0, item_len >= 1");
    NSD_REQUIRE(plan && item_ptr, "null pointer");
    NSD_REQUIRE(nseg == 0 || (segptr && long_seg && long_first && huge_idx && chunk_item &&
                              chunk_ord && empty_seg && ws),
                "null pointer");
    if (2LL * nnz + nseg >= (1LL << 31)) return fail(NSD_ERR_TOO_LARGE, "plan cost overflows int32");
    hipStream_t st = as_stream(stream);
    *plan = nsd_plan{};
    plan->item_len = item_len;
    plan->item_ptr = item_ptr;
    plan->long_seg = long_seg;
    plan->long_first = long_first;
    plan->huge_idx = huge_idx;
    plan->chunk_item = chunk_item;
    plan->chunk_ord = chunk_ord;
    plan->empty_seg = empty_seg;
    if (nseg == 0) {
        plan_sentinel_kernel<<<1, 1, 0, st>>>(item_ptr, 0);
        NSD_TRY(check_launch("plan_sentinel_kernel"));
        NSD_HIP(hipStreamSynchronize(st));
        return NSD_OK;
    }
    if (ws_bytes < plan_ws_bytes())
        return fail(NSD_ERR_WORKSPACE, "workspace %zu < %zu", ws_bytes, plan_ws_bytes());
    Carver c(ws);
    PlanCost *costs = c.take<PlanCost>(kPlanMaxBlocks);
    PlanCounts *counts = c.take<PlanCounts>(kPlanMaxBlocks);
    int32_t *longest = c.take<int32_t>(kPlanMaxBlocks);
    int32_t *tot = c.take<int32_t>(64);  // the counts, then the longest's chunks
    const int64_t per = plan_per_block(nseg);
    const unsigned g = (unsigned)ceil_div(nseg, per);

    plan_cost_kernel<<<g, kPlanThreads, 0, st>>>(nseg, per, segptr, item_len, costs);
    NSD_TRY(check_launch("plan_cost_kernel"));
    plan_count_kernel<<<g, kPlanThreads, 0, st>>>(nseg, per, segptr, item_len, costs, counts,
                                                  longest);
    NSD_TRY(check_launch("plan_count_kernel"));
    PlanOut out{item_ptr, long_seg, long_first, huge_idx, chunk_item, chunk_ord, empty_seg};
    plan_fill_kernel<<<g, kPlanThreads, 0, st>>>(nseg, nnz, per, segptr, item_len, costs, counts,
                                                 longest, out, tot);
    NSD_TRY(check_launch("plan_fill_kernel"));
    int32_t h[kPlanCounts + 1];
    NSD_HIP(hipMemcpyAsync(h, tot, sizeof(h), hipMemcpyDeviceToHost, st));
    NSD_HIP(hipStreamSynchronize(st));
    plan->nitems = h[0];
    plan->nlong = h[1];
    plan->nempty = h[2];
    plan->nchunks = h[3];
    plan->nhuge = h[4];
    plan->longest_chunks = h[5];
    return NSD_OK;
}

}  // extern "C"
