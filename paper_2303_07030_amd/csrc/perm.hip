// A fixed permutation of fp32 values applied in two coalesced passes:
//   dst[q] = src[perm[q]]   for q < n
// (the values of a sparse operand between its CSR and CSC orders, and a
// sparse gradient back; both directions are permutations of this form).
//
// A direct gather reads one 4-byte value per random cache line.  Here the
// permutation is split, once per pattern, into two local ones of bounded
// span (a two-digit radix permutation), so every global access is a whole
// line or a run of consecutive values:
//   pass 1, per source tile of T consecutive elements: the tile is staged in
//     LDS and written out in the order of its elements' destination buckets
//     (B = T consecutive destinations each), one run per bucket, into a
//     staging array whose bucket d occupies [d T, (d + 1) T) and holds its
//     elements by source tile;
//   pass 2, per destination bucket: the bucket's staging run is read
//     contiguously, placed in LDS at its local destination offsets, and the
//     bucket is written out contiguously.
// The plan stores, per element, the staging position and the local source
// index of pass 1's output slots, and the local destination offset of the
// staging slots (16-bit local indices: T = 2^15).  It is built by one
// partition of the permutation (below).  The result is an exact copy (bit
// for bit).
#include <algorithm>

#include "nsd_internal.hpp"

namespace nsd {

constexpr int kPermThreads = 1024;
constexpr int kPermBits = 15;              // log2 of the tile: a local index inside it
constexpr int kPermTile = 1 << kPermBits;  // T = B, the LDS span of either pass (128 KiB)

static int64_t perm_tiles(int64_t n) { return ceil_div(n, kPermTile); }

// ------------------------------------------------------------- apply

// Each thread handles kPermPer elements of its tile, strided by the block
// size, in batches of kPermBatch whose loads are all issued before any is
// used (one memory round trip per batch, not per element).  Everything read
// is read once and the result written once: those accesses are
// non-temporal, leaving the L2 to the staging runs of pass 1, which meet
// there with their neighbours' (measured on MI355X, a move of 60M values:
// 0.310 ms with ordinary accesses, 0.266 ms so; the staging stores made
// non-temporal as well, 0.433 ms).
constexpr int kPermPer = kPermTile / kPermThreads;
constexpr int kPermBatch = 8;
static_assert(kPermPer % kPermBatch == 0, "whole batches per thread");

__global__ __launch_bounds__(kPermThreads) void perm_pass1_kernel(int64_t n, const float *src,
                                                                  const int32_t *stage,
                                                                  const uint16_t *src_local,
                                                                  float *staging) {
    __shared__ float tile[kPermTile];
    const int64_t t0 = xcd_contiguous_tile() * kPermTile;
    const int len = (int)min((int64_t)kPermTile, n - t0);
    const int tid = threadIdx.x;
    for (int b = 0; b < kPermPer; b += kPermBatch) {
        float v[kPermBatch];
#pragma unroll
        for (int u = 0; u < kPermBatch; ++u) {
            const int i = tid + (b + u) * kPermThreads;
            v[u] = i < len ? __builtin_nontemporal_load(src + t0 + i) : 0.f;
        }
#pragma unroll
        for (int u = 0; u < kPermBatch; ++u) tile[tid + (b + u) * kPermThreads] = v[u];
    }
    __syncthreads();
    for (int b = 0; b < kPermPer; b += kPermBatch) {
        int32_t st[kPermBatch];
        int loc[kPermBatch];
#pragma unroll
        for (int u = 0; u < kPermBatch; ++u) {
            const int o = tid + (b + u) * kPermThreads;
            st[u] = o < len ? __builtin_nontemporal_load(stage + t0 + o) : -1;
            loc[u] = o < len ? __builtin_nontemporal_load(src_local + t0 + o) : 0;
        }
#pragma unroll
        for (int u = 0; u < kPermBatch; ++u)
            if (st[u] >= 0) staging[st[u]] = tile[loc[u]];
    }
}

__global__ __launch_bounds__(kPermThreads) void perm_pass2_kernel(int64_t n,
                                                                  const float *staging,
                                                                  const uint16_t *dst_local,
                                                                  float *dst) {
    __shared__ float bucket[kPermTile];
    const int64_t d0 = (int64_t)blockIdx.x * kPermTile;
    const int len = (int)min((int64_t)kPermTile, n - d0);
    const int tid = threadIdx.x;
    for (int b = 0; b < kPermPer; b += kPermBatch) {
        float v[kPermBatch];
        int loc[kPermBatch];
#pragma unroll
        for (int u = 0; u < kPermBatch; ++u) {
            const int s = tid + (b + u) * kPermThreads;
            v[u] = s < len ? __builtin_nontemporal_load(staging + d0 + s) : 0.f;
            loc[u] = s < len ? __builtin_nontemporal_load(dst_local + d0 + s) : -1;
        }
#pragma unroll
        for (int u = 0; u < kPermBatch; ++u)
            if (loc[u] >= 0) bucket[loc[u]] = v[u];
    }
    __syncthreads();
    for (int b = 0; b < kPermPer; b += kPermBatch) {
#pragma unroll
        for (int u = 0; u < kPermBatch; ++u) {
            const int i = tid + (b + u) * kPermThreads;
            if (i < len) __builtin_nontemporal_store(bucket[i], dst + d0 + i);
        }
    }
}

// ------------------------------------------------------------- build

// A plan is one partition of the given array.  key[i] is the far end of the
// move of near index i: the destination of source i (inverse), or the source
// of destination i.  Near indices come in tiles of T, far indices in windows
// of T; the elements of tile t whose far end lies in window f form one run
// (t, f), in near order.  Near side, tile t holds its runs by f; far side,
// window f holds its runs by t: these two orders are the slots of pass 1 and
// of the staging array (which is which depends on the direction).
//   hist:  counts of every run, [f][t];  its exclusive scan is the far-side
//          position of every run;
//   sort:  per tile, the elements sorted by window in LDS, then both sides'
//          entries written: the near side's in order, the far side's in runs;
//   check: the far ends are distinct (a bitmap per window) and every window
//          full, so the given array is a permutation.
// The moves in both directions have the same runs and local offsets; only
// their slots' staging positions differ (the near side's slot to the far
// side's, or back), so one partition makes both plans: two of 50M elements
// 1.73 -> 0.92 ms on MI355X.

constexpr int kPermWaves = kPermThreads / kWave;

// A far index as counted and placed: out of range ones (reported through
// the flag) count as the last, so every write stays inside its array.
__device__ __forceinline__ uint32_t perm_far(int32_t k, int64_t n) {
    const uint32_t last = (uint32_t)(n - 1);
    return (uint32_t)k < last ? (uint32_t)k : last;
}

// Counts of tile t's elements per window, two 16-bit counters to an LDS word
// (at most T = 2^15 elements each); [0] of the dynamic LDS on.
__global__ __launch_bounds__(kPermThreads) void perm_hist_kernel(int64_t n, const int32_t *key,
                                                                 int32_t ntiles, int32_t *hist,
                                                                 int32_t *flag) {
    extern __shared__ uint32_t wcount[];
    const int64_t t = blockIdx.x, t0 = t * kPermTile;
    const int len = (int)min((int64_t)kPermTile, n - t0);
    for (int i = threadIdx.x; i < (ntiles + 1) / 2; i += kPermThreads) wcount[i] = 0;
    __syncthreads();
    bool bad = false;
    for (int b = 0; b < kPermPer; b += kPermBatch) {
        int32_t k[kPermBatch];
#pragma unroll
        for (int u = 0; u < kPermBatch; ++u) {
            const int i = (int)threadIdx.x + (b + u) * kPermThreads;
            k[u] = i < len ? key[t0 + i] : 0;
        }
#pragma unroll
        for (int u = 0; u < kPermBatch; ++u) {
            const int i = (int)threadIdx.x + (b + u) * kPermThreads;
            if (i < len) {
                bad = bad || k[u] < 0 || k[u] >= n;
                const uint32_t f = perm_far(k[u], n) >> kPermBits;
                atomicAdd(&wcount[f >> 1], 1u << ((f & 1) * 16));
            }
        }
    }
    if (__ballot(bad) && (threadIdx.x & (kWave - 1)) == 0) atomicOr(flag, 1);
    __syncthreads();
    for (int f = threadIdx.x; f < ntiles; f += kPermThreads)
        hist[(int64_t)f * ntiles + t] = (int32_t)((wcount[f >> 1] >> ((f & 1) * 16)) & 0xffffu);
}

// Keeps the compiler from moving work across every fourth unrolled round: it
// hoists all rounds' loads otherwise and spills (128 registers a thread in a
// block of 1024).
__device__ __forceinline__ void perm_keep_order(int i) {
    if (i % 4 == 3) __builtin_amdgcn_sched_barrier(0);
}

// Tile t sorted by window and written out.  The words (window << 15 | near
// offset) are sorted by their window bits in LDS, 8 bits a pass, stably: a
// wave owns 2048 consecutive words, 32 rounds of 64; a round's equal digits
// are matched with ballots, and a word's rank is the count of its digit in
// the wave's earlier rounds and below it in the round.  Bound by the ranking
// and by the far side's short runs (T^2 / n elements, 21 of 50M).
__global__ __launch_bounds__(kPermThreads) void perm_sort_kernel(
    int64_t n, const int32_t *key, int32_t ntiles, int window_bits, const int32_t *run_pos,
    uint16_t *near_local, uint16_t *far_local, int32_t *near_stage, int32_t *far_stage) {
    __shared__ uint32_t tile[kPermTile];
    __shared__ uint32_t wcnt[kPermWaves][256];
    __shared__ uint32_t dstart[256];
    const int64_t t = xcd_contiguous_tile(), t0 = t * kPermTile;
    const int len = (int)min((int64_t)kPermTile, n - t0);
    const int tid = threadIdx.x, lane = tid & (kWave - 1), wave = tid / kWave;
    const int wbase = wave * (kPermPer * kWave);
    int first = wbase + lane;  // this lane's word of round 0
    // the tile's own slices: 32-bit offsets from them keep addresses out of
    // the vector registers
    const int32_t *tkey = key + t0;
    uint16_t *tlocal = near_local + t0;
    int32_t *tstage = near_stage + t0;  // used when not NULL
    const int32_t *tpos = run_pos + t;
    uint32_t v[kPermPer];
#pragma unroll
    for (int i = 0; i < kPermPer; ++i) {
        const int p = first + i * kWave;
        // past the end: above every word, so they stay last
        v[i] = p < len ? ((perm_far(tkey[p], n) >> kPermBits) << kPermBits) | (uint32_t)p : ~0u;
    }
    for (int sh = kPermBits; sh < kPermBits + window_bits; sh += 8) {
        for (int i = tid; i < kPermWaves * 256; i += kPermThreads) (&wcnt[0][0])[i] = 0;
        __syncthreads();
        uint32_t rank[kPermPer / 2];  // two 16-bit ranks (below 2048) to a register
#pragma unroll
        for (int i = 0; i < kPermPer; ++i) {
            const uint32_t d = (v[i] >> sh) & 255u;
            uint64_t same = ~0ull;
#pragma unroll
            for (int b = 0; b < 8; ++b) {
                const bool bit = (d >> b) & 1;
                const uint64_t m = __ballot(bit);
                same &= bit ? m : ~m;
            }
            const int below = __popcll(same & __lanemask_lt());
            const uint32_t prev = wcnt[wave][d];
            if (i % 2 == 0) rank[i / 2] = prev + below;
            else rank[i / 2] |= (prev + below) << 16;
            __builtin_amdgcn_wave_barrier();
            if (below == 0) wcnt[wave][d] = prev + __popcll(same);
            __builtin_amdgcn_wave_barrier();
            perm_keep_order(i);
        }
        __syncthreads();
        uint32_t total = 0;
        if (tid < 256) {  // the waves' offsets inside each digit's run
            for (int w = 0; w < kPermWaves; ++w) {
                const uint32_t c = wcnt[w][tid];
                wcnt[w][tid] = total;
                total += c;
            }
            dstart[tid] = total;
        }
        __syncthreads();
        for (int off = 1; off < 256; off <<= 1) {  // the runs' starts: a scan over the digits
            const uint32_t add = tid < 256 && tid >= off ? dstart[tid - off] : 0;
            __syncthreads();
            if (tid < 256) dstart[tid] += add;
            __syncthreads();
        }
        if (tid < 256) dstart[tid] -= total;
        __syncthreads();
        int shift = sh;
        opaque(shift);
#pragma unroll
        for (int i = 0; i < kPermPer; ++i) {
            const uint32_t d = (v[i] >> shift) & 255u;
            tile[dstart[d] + wcnt[wave][d] + ((rank[i / 2] >> (i % 2 * 16)) & 0xffffu)] = v[i];
            perm_keep_order(i);
        }
        __syncthreads();
        opaque(first);
#pragma unroll
        for (int i = 0; i < kPermPer; ++i) v[i] = tile[first + i * kWave];
    }
    if (window_bits == 0) {
#pragma unroll
        for (int i = 0; i < kPermPer; ++i) tile[first + i * kWave] = v[i];
    }
    __syncthreads();
    // the run holding each word: its first slot is the last window change at
    // or before it.  A wave finds that of its first word by bisection, the
    // others by ballots as it goes along.
    const uint32_t w0 = tile[wbase] >> kPermBits;
    int lo = 0, hi = wbase;  // first slot of window w0
    while (lo < hi) {
        const int mid = (lo + hi) >> 1;
        if ((tile[mid] >> kPermBits) < w0) lo = mid + 1;
        else hi = mid;
    }
    int open = lo;
    opaque(first);
    int32_t far[kPermPer];
#pragma unroll
    for (int i = 0; i < kPermPer; ++i) {
        const int o = first + i * kWave;
        const uint32_t f = v[i] >> kPermBits;
        const bool head = o > 0 && (tile[o - 1] >> kPermBits) != f;
        const uint64_t heads = __ballot(head);
        const uint64_t mine = heads & (__lanemask_lt() | (1ull << lane));
        const int start = mine ? wbase + i * kWave + 63 - __clzll((long long)mine) : open;
        if (heads) open = wbase + i * kWave + 63 - __clzll((long long)heads);
        far[i] = -1;
        if (o < len) {
            far[i] = tpos[(int64_t)f * ntiles] + (o - start);
            tlocal[o] = (uint16_t)(v[i] & (kPermTile - 1));
            if (near_stage) tstage[o] = far[i];
            if (far_stage) far_stage[far[i]] = (int32_t)t0 + o;
        }
        perm_keep_order(i);
    }
    __syncthreads();
    // the far ends' offsets in their windows, by near offset, then by slot
    opaque(first);
    uint16_t *low = reinterpret_cast<uint16_t *>(tile);
#pragma unroll
    for (int i = 0; i < kPermPer; ++i) {
        const int p = first + i * kWave;
        if (p < len) low[p] = (uint16_t)(perm_far(tkey[p], n) & (kPermTile - 1));
        perm_keep_order(i);
    }
    __syncthreads();
#pragma unroll
    for (int i = 0; i < kPermPer; ++i) {
        if (far[i] >= 0) far_local[far[i]] = low[v[i] & (kPermTile - 1)];
        perm_keep_order(i);
    }
}

// Window f holds T far ends (the last one what is left), all different.
__global__ __launch_bounds__(kPermThreads) void perm_check_kernel(int64_t n, int32_t ntiles,
                                                                  const int32_t *run_pos,
                                                                  const uint16_t *far_local,
                                                                  int32_t *flag) {
    __shared__ uint32_t seen[kPermTile / 32];
    const int64_t f = blockIdx.x, f0 = f * kPermTile;
    const int len = (int)min((int64_t)kPermTile, n - f0);
    for (int i = threadIdx.x; i < kPermTile / 32; i += kPermThreads) seen[i] = 0;
    __syncthreads();
    bool bad = run_pos[f * ntiles] != f0;
    for (int i = threadIdx.x; i < len; i += kPermThreads) {
        const uint32_t q = far_local[f0 + i];
        const uint32_t bit = 1u << (q & 31);
        bad = bad || (atomicOr(&seen[q >> 5], bit) & bit) != 0;
    }
    if (__ballot(bad) && (threadIdx.x & (kWave - 1)) == 0) atomicOr(flag, 2);
}

static size_t perm_build_ws(int64_t n) {
    Carver c(nullptr);
    const int64_t nt = perm_tiles(std::max<int64_t>(n, 1));
    c.take<int32_t>(64);
    c.take<int32_t>(nt * nt);
    return c.bytes() + scan_ws_bytes(nt * nt);
}

static nsd_perm_plan perm_plan_of(int32_t n, const int32_t *stage, const uint16_t *src_local,
                                  const uint16_t *dst_local) {
    nsd_perm_plan p{};
    p.n = n;
    p.tile = kPermTile;
    p.stage = stage;
    p.src_local = src_local;
    p.dst_local = dst_local;
    return p;
}

// The partition of perm and its check; near_stage and far_stage: the staging
// position of each near slot on the far side, and of each far slot on the
// near side (either may be NULL).
static nsd_status perm_partition(int32_t n, const int32_t *perm, uint16_t *near_local,
                                 uint16_t *far_local, int32_t *near_stage, int32_t *far_stage,
                                 void *ws, size_t ws_bytes, hipStream_t st) {
    if (n == 0) return NSD_OK;
    const size_t need = perm_build_ws(n);
    if (ws_bytes < need) return fail(NSD_ERR_WORKSPACE, "workspace %zu < %zu", ws_bytes, need);
    const int64_t nt = perm_tiles(n);
    Carver c(ws);
    int32_t *flag = c.take<int32_t>(64);
    int32_t *runs = c.take<int32_t>(nt * nt);
    void *scan_ws = c.base + c.bytes();
    int window_bits = 0;
    while ((int64_t(1) << window_bits) < nt) ++window_bits;
    NSD_HIP(hipMemsetAsync(flag, 0, sizeof(int32_t), st));
    perm_hist_kernel<<<(unsigned)nt, kPermThreads, (size_t)((nt + 1) / 2) * sizeof(uint32_t), st>>>(
        n, perm, (int32_t)nt, runs, flag);
    NSD_TRY(check_launch("perm_hist_kernel"));
    NSD_TRY(scan_exclusive(runs, runs, nt * nt, nullptr, scan_ws, st));
    perm_sort_kernel<<<(unsigned)nt, kPermThreads, 0, st>>>(n, perm, (int32_t)nt, window_bits, runs,
                                                            near_local, far_local, near_stage,
                                                            far_stage);
    NSD_TRY(check_launch("perm_sort_kernel"));
    perm_check_kernel<<<(unsigned)nt, kPermThreads, 0, st>>>(n, (int32_t)nt, runs, far_local, flag);
    NSD_TRY(check_launch("perm_check_kernel"));
    int32_t h = 0;
    NSD_HIP(hipMemcpyAsync(&h, flag, sizeof(int32_t), hipMemcpyDeviceToHost, st));
    NSD_HIP(hipStreamSynchronize(st));
    if (h) return fail(NSD_ERR_BAD_FORMAT, "not a permutation of [0, %d)", n);
    return NSD_OK;
}

}  // namespace nsd

using namespace nsd;

extern "C" {

nsd_status nsd_perm_plan_workspace_size(int32_t n, size_t *bytes) {
    NSD_REQUIRE(bytes != nullptr, "bytes is NULL");
    NSD_REQUIRE(n >= 0, "negative length");
    *bytes = perm_build_ws(n);
    return NSD_OK;
}

nsd_status nsd_perm_plan_build(int32_t n, const int32_t *perm, int inverse, int32_t *stage,
                               uint16_t *src_local, uint16_t *dst_local, nsd_perm_plan *plan,
                               void *ws, size_t ws_bytes, void *stream) {
    NSD_REQUIRE(n >= 0 && plan != nullptr, "negative length or NULL plan");
    NSD_REQUIRE(n == 0 || (perm && stage && src_local && dst_local && ws), "null pointer");
    *plan = perm_plan_of(n, stage, src_local, dst_local);
    // dst[perm[q]] = src[q] (inverse): near indices are sources; dst[q] =
    // src[perm[q]]: they are destinations
    return perm_partition(n, perm, inverse ? src_local : dst_local,
                          inverse ? dst_local : src_local, inverse ? stage : nullptr,
                          inverse ? nullptr : stage, ws, ws_bytes, as_stream(stream));
}

nsd_status nsd_perm_plan_build_pair(int32_t n, const int32_t *perm, int32_t *stage,
                                    int32_t *inv_stage, uint16_t *near_local,
                                    uint16_t *far_local, nsd_perm_plan *plan,
                                    nsd_perm_plan *inv_plan, void *ws, size_t ws_bytes,
                                    void *stream) {
    NSD_REQUIRE(n >= 0 && plan != nullptr && inv_plan != nullptr, "negative length or NULL plan");
    NSD_REQUIRE(n == 0 || (perm && stage && inv_stage && near_local && far_local && ws),
                "null pointer");
    *plan = perm_plan_of(n, stage, far_local, near_local);
    *inv_plan = perm_plan_of(n, inv_stage, near_local, far_local);
    return perm_partition(n, perm, near_local, far_local, inv_stage, stage, ws, ws_bytes,
                          as_stream(stream));
}

nsd_status nsd_permute_f32(const nsd_perm_plan *plan, const float *src, float *dst,
                           float *staging, void *stream) {
    NSD_REQUIRE(plan != nullptr, "plan is NULL");
    NSD_REQUIRE(plan->n >= 0, "negative length");
    if (plan->n == 0) return NSD_OK;
    NSD_REQUIRE(plan->tile == kPermTile, "plan built with tile %d, library uses %d", plan->tile,
                kPermTile);
    NSD_REQUIRE(plan->stage && plan->src_local && plan->dst_local, "plan is not built");
    NSD_REQUIRE(src && dst && staging, "null pointer");
    NSD_REQUIRE(src != dst, "src and dst must not alias");
    hipStream_t st = as_stream(stream);
    const unsigned nt = (unsigned)perm_tiles(plan->n);
    probe_begin(NSD_KERNEL_PERM, st);
    perm_pass1_kernel<<<nt, kPermThreads, 0, st>>>(plan->n, src, plan->stage, plan->src_local,
                                                   staging);
    NSD_TRY(check_launch("perm_pass1_kernel"));
    perm_pass2_kernel<<<nt, kPermThreads, 0, st>>>(plan->n, staging, plan->dst_local, dst);
    probe_end(NSD_KERNEL_PERM, st);
    return check_launch("perm_pass2_kernel");
}

}  // extern "C"
