// Passes of dense width 1: SpMV, its transpose, their vector-Jacobian
// products, column sums and the SMVM loss.
//
// With one column there is no dense row to spread over lanes: an entry is a
// few words, and the pass is bound by streaming them.  A slot per work item
// (one lane walking its own 16 to 48 consecutive entries) made every load of
// a wave touch 64 lines, and the SMVM loss of 20M entries took 0.90 ms on
// MI355X (its floor: 0.05).  Here a
// block takes one tile of consecutive entries whatever segments they belong
// to, every thread E consecutive ones (16-byte loads), and the segment sums
// are a segmented scan: in the thread, over the wave's lanes, over the block's
// waves.  A segment inside one tile is written directly; one that crosses
// tiles leaves its first tile's part in tail[] and each later tile's in
// head[], added in tile order by the combine, or is finished by the block in
// which it starts (vec1_run says when).  Everything is summed in a fixed order,
// so results are the same from run to run.  The SMVM loss of 20M
// entries takes 0.26 ms: 0.13 the sampled product (20M gathers of a word of x,
// a 128-byte line from L2 each: the L2's rate), 0.09 the values' move to CSC
// order, 0.03 their sums (5.4 TB/s).
#include "nsd_internal.hpp"
#include "segreduce.hpp"
#include "segreduce_dev.hpp"

namespace nsd {

struct Vec1Params {
    SgrParams s;                 // part: unused
    const float *own = nullptr;  // [nseg]: DUAL only
    float *sdd = nullptr;        // sampled products at the weights' positions
    float sdd_alpha = 1.f;
    double *loss_part = nullptr; // one per tile (NULL: no loss)
    double *loss = nullptr;      // WHOLE: the loss, by the first block over `entries`
    SddmmParams entries;         // the operand's entries in their own order (WHOLE)
    float *head = nullptr, *tail = nullptr;  // [tiles]
};

// E words from p, 16 bytes a load where E allows (p aligned to words only).
template <int E, class T>
__device__ __forceinline__ void load_words(const T *p, T (&v)[E]) {
    if constexpr (E % 4 == 0) {
        typedef T T4 __attribute__((ext_vector_type(4), aligned(4)));
#pragma unroll
        for (int i = 0; i < E; i += 4) {
            const T4 t = *reinterpret_cast<const T4 *>(p + i);
            v[i] = t.x;
            v[i + 1] = t.y;
            v[i + 2] = t.z;
            v[i + 3] = t.w;
        }
    } else {
#pragma unroll
        for (int i = 0; i < E; ++i) v[i] = p[i];
    }
}

template <int E>
__device__ __forceinline__ void store_words(float *p, const float (&v)[E]) {
    if constexpr (E % 4 == 0) {
        typedef float f4 __attribute__((ext_vector_type(4), aligned(4)));
#pragma unroll
        for (int i = 0; i < E; i += 4) {
            const f4 t = {v[i], v[i + 1], v[i + 2], v[i + 3]};
            *reinterpret_cast<f4 *>(p + i) = t;
        }
    } else {
#pragma unroll
        for (int i = 0; i < E; ++i) p[i] = v[i];
    }
}

// Block total of per-lane fp64 values over NW waves, in a fixed order; valid
// in thread 0.
template <int NW>
__device__ __forceinline__ double block_total(double v) {
    __shared__ double wsum[NW];
#pragma unroll
    for (int m = kWave / 2; m >= 1; m >>= 1) v += __shfl_xor(v, m, kWave);
    if (threadIdx.x % kWave == 0) wsum[threadIdx.x / kWave] = v;
    __syncthreads();
    double t = 0.0;
#pragma unroll
    for (int i = 0; i < NW; ++i) t += wsum[i];
    return t;
}

// The loss of a small pass by one block, entry by entry in the operand's own
// order: sum w_p X[row_p] Y[col_p] (X NULL: ones).
template <int T>
__device__ __forceinline__ void vec1_small_loss(const SddmmParams &a, double *loss) {
    constexpr int kDeep = 8;  // loads in flight per thread
    double s = 0.0;
    for (int p0 = threadIdx.x; p0 < a.nnz; p0 += T * kDeep) {
        float d[kDeep], w[kDeep];
        int c[kDeep], r[kDeep];
#pragma unroll
        for (int u = 0; u < kDeep; ++u) {
            const int p = min(p0 + u * T, a.nnz - 1);
            c[u] = a.colind[p];
            r[u] = a.X ? a.rowidx[p] : 0;
            w[u] = a.w[p];
        }
#pragma unroll
        for (int u = 0; u < kDeep; ++u) d[u] = a.Y[c[u]] * (a.X ? a.X[r[u]] : 1.f);
#pragma unroll
        for (int u = 0; u < kDeep; ++u)
            if (p0 + u * T < a.nnz) s += (double)w[u] * (double)d[u];
    }
    const double t = block_total<T / kWave>(s);
    if (threadIdx.x == 0) *loss = t;
}

// One tile of T * E entries per block; blocks past the tiles zero the empty
// segments.  A WHOLE pass is complete in this launch: the block in which a
// segment starts also adds its entries past the tile, and the loss (of tiles of
// one entry per thread) is one more block, the first.  out[s] = alpha sum w_p X[idx_p]; with DUAL also
// sdd[pos_p] = sdd_alpha own[s] X[idx_p] and the loss sum w_p own[s] X[idx_p].
template <int T, int E, bool DUAL, bool WHOLE>
__global__ __launch_bounds__(T) void vec1_kernel(Vec1Params f) {
    constexpr int kTile = T * E, kWaves = T / kWave;
    const SgrParams &a = f.s;
    const int tid = threadIdx.x;
    int blk = blockIdx.x;
    if constexpr (WHOLE && DUAL && E == 1) {
        if (f.loss && blk-- == 0) {
            vec1_small_loss<T>(f.entries, f.loss);
            return;
        }
    }
    if (blk >= a.item_blocks) {
        const int64_t e = (int64_t)(blk - a.item_blocks) * T + tid;
        if (e < a.plan.nempty) a.out[a.plan.empty_seg[e]] = 0.f;
        return;
    }
    const int64_t n = a.nnz, p0 = (int64_t)blk * kTile + (int64_t)tid * E;
    int r[E], c[E], pos[E];  // segment (-1: past the end), gathered row, weight position
    float w[E], x[E];
    if (p0 + E <= n) {
        load_words<E>(a.segidx + p0, r);
        if (a.X) load_words<E>(a.idx + p0, c);
        if (a.wperm) {
            load_words<E>(a.wperm + p0, pos);
#pragma unroll
            for (int u = 0; u < E; ++u) w[u] = a.w[pos[u]];
        } else if (a.w) {
            load_words<E>(a.w + p0, w);
        }
    } else {
#pragma unroll
        for (int u = 0; u < E; ++u) {
            const bool in = p0 + u < n;
            r[u] = in ? a.segidx[p0 + u] : -1;
            c[u] = in && a.X ? a.idx[p0 + u] : 0;
            pos[u] = in && a.wperm ? a.wperm[p0 + u] : 0;
            w[u] = in && a.w ? a.w[a.wperm ? (int64_t)pos[u] : p0 + u] : 0.f;
        }
    }
#pragma unroll
    for (int u = 0; u < E; ++u) {
        x[u] = a.X ? a.X[c[u]] : 1.f;
        if (!a.w) w[u] = 1.f;
    }
    double lsum = 0.0;
    if constexpr (DUAL) {
        float d[E];
#pragma unroll
        for (int u = 0; u < E; ++u) {
            d[u] = r[u] >= 0 ? f.own[r[u]] * x[u] : 0.f;
            if (r[u] >= 0) lsum += (double)w[u] * d[u];
            d[u] *= f.sdd_alpha;
        }
        if (f.sdd) {
            if (a.wperm) {
#pragma unroll
                for (int u = 0; u < E; ++u)
                    if (r[u] >= 0) f.sdd[pos[u]] = d[u];
            } else if (p0 + E <= n) {
                store_words<E>(f.sdd + p0, d);
            } else {
#pragma unroll
                for (int u = 0; u < E; ++u)
                    if (r[u] >= 0) f.sdd[p0 + u] = d[u];
            }
        }
    }
    // the thread's runs: the first one's sum, whole ones in between written,
    // the last one's sum
    float run = r[0] >= 0 ? w[0] * x[0] : 0.f, first = 0.f;
    bool single = true;
#pragma unroll
    for (int u = 1; u < E; ++u) {
        const float v = r[u] >= 0 ? w[u] * x[u] : 0.f;
        if (r[u] != r[u - 1]) {
            if (single) first = run;
            else a.out[r[u - 1]] = a.alpha * run;
            single = false;
            run = v;
        } else {
            run += v;
        }
    }
    const int lane = tid & (kWave - 1), wave = tid / kWave;
    int prev = __shfl_up(r[E - 1], 1, kWave), next = __shfl_down(r[0], 1, kWave);
    if (lane == 0) prev = p0 > 0 && p0 <= n ? a.segidx[p0 - 1] : -1;
    if (lane == kWave - 1) next = p0 + E < n ? a.segidx[p0 + E] : -1;
    // sum of the run open at each lane's end, back to the wave's start; starts:
    // it starts inside the wave
    float sum = run;
    bool starts = !single || prev != r[0];
#pragma unroll
    for (int d = 1; d < kWave; d <<= 1) {
        const float y = __shfl_up(sum, d, kWave);
        const bool ys = __shfl_up((int)starts, d, kWave) != 0;
        if (lane >= d) {
            if (!starts) sum += y;
            starts = starts || ys;
        }
    }
    __shared__ float wsum[kWaves];
    __shared__ int wstarts[kWaves];
    if (lane == kWave - 1) {
        wsum[wave] = sum;
        wstarts[wave] = starts;
    }
    __syncthreads();
    // the run open at the end of the wave before: its sum inside the tile, and
    // whether it starts in it
    float carry = 0.f;
    bool in_tile = false;
    for (int i = 0; i < wave; ++i) {
        carry = wstarts[i] ? wsum[i] : carry + wsum[i];
        in_tile = in_tile || wstarts[i];
    }
    float before = __shfl_up(sum, 1, kWave);
    bool before_starts = __shfl_up((int)starts, 1, kWave) != 0;
    if (lane == 0) {
        before = 0.f;
        before_starts = false;
    }
    // (a WHOLE pass drops the parts of segments that start in earlier tiles)
    if (!single && r[0] >= 0) {  // the first run ends in this thread
        const bool goes_on = prev == r[0];
        const float t = !goes_on ? first : (before_starts ? before : before + carry) + first;
        if (!goes_on || before_starts || in_tile) a.out[r[0]] = a.alpha * t;
        else if (!WHOLE) f.head[blk] = t;
    }
    __shared__ float tail;
    __shared__ int tail_seg;
    if (WHOLE && tid == T - 1) tail_seg = -1;
    if (r[E - 1] >= 0) {
        const float t = starts ? sum : sum + carry;
        const bool here = starts || in_tile;
        if (next != r[E - 1]) {  // the last run ends with this thread
            if (here) a.out[r[E - 1]] = a.alpha * t;
            else if (!WHOLE) f.head[blk] = t;
        } else if (tid == T - 1) {  // or goes on in the next tile
            if (WHOLE) {
                tail = t;
                tail_seg = here ? r[E - 1] : -1;
            } else {
                if (here) f.tail[blk] = t;
                else f.head[blk] = t;
            }
        }
    }
    if constexpr (WHOLE) {
        __syncthreads();
        if (tail_seg >= 0) {  // the rest of the segment open at the tile's end
            float s = 0.f;
            const int64_t end = a.segptr[tail_seg + 1];
            for (int64_t p = (int64_t)(blk + 1) * kTile + tid; p < end; p += T)
                s += (a.w ? a.w[a.wperm ? (int64_t)a.wperm[p] : p] : 1.f) *
                     (a.X ? a.X[a.idx[p]] : 1.f);
#pragma unroll
            for (int m = kWave / 2; m >= 1; m >>= 1) s += __shfl_xor(s, m, kWave);
            __syncthreads();  // wsum has been read
            if (lane == 0) wsum[wave] = s;
            __syncthreads();
            if (tid == 0) {
                float t = tail;
                for (int i = 0; i < kWaves; ++i) t += wsum[i];
                a.out[tail_seg] = a.alpha * t;
            }
        }
        return;
    }
    if constexpr (DUAL) {
        if (f.loss_part) {
            const double t = block_total<kWaves>(lsum);
            if (tid == 0) f.loss_part[blk] = t;
        }
    }
}

// Segments that cross tiles, one wave per tile: the one that starts in tile b
// and goes on takes tail[b] and the head[] of every tile it reaches.  The last
// block is the loss total (when there is a job).
__global__ __launch_bounds__(kBlock) void vec1_fix_kernel(Vec1Params f, int64_t tile,
                                                          LossJob job) {
    if (job.loss && blockIdx.x == gridDim.x - 1) {
        loss_total_block<kFixSumChains>(job);
        return;
    }
    const SgrParams &a = f.s;
    const int lane = threadIdx.x & (kWave - 1);
    const int64_t b = (int64_t)blockIdx.x * kBlockWaves + threadIdx.x / kWave;
    if (b >= a.item_blocks - 1) return;
    const int64_t e = (b + 1) * tile;
    const int seg = a.segidx[e - 1];
    if (a.segidx[e] != seg || a.segptr[seg] < b * tile) return;
    const int64_t last = ((int64_t)a.segptr[seg + 1] - 1) / tile;
    float s = b + 1 + lane <= last ? f.head[b + 1 + lane] : 0.f;
    // a segment of many tiles: independent loads (a column of 50M entries has
    // 24K heads, 121 us with one load in flight at a time, 23 so)
    constexpr int kDeep = 16;
    for (int64_t j0 = b + 1 + kWave + lane; j0 <= last; j0 += kDeep * kWave) {
        float x[kDeep];
#pragma unroll
        for (int u = 0; u < kDeep; ++u) x[u] = f.head[min(j0 + u * kWave, last)];
#pragma unroll
        for (int u = 0; u < kDeep; ++u)
            if (j0 + u * kWave <= last) s += x[u];
    }
#pragma unroll
    for (int m = kWave / 2; m >= 1; m >>= 1) s += __shfl_xor(s, m, kWave);
    if (lane == 0) a.out[seg] = a.alpha * (f.tail[b] + s);
}

// Tiles of one pass.  A small one is complete in one launch: a combine and
// its launch cost more than re-reading the crossing segments, unless one block
// has more than kVec1Tail entries of a segment to add, twice as many if it
// gathers nothing for them (a row of 16K entries 10.5 us, with the combine 5.1), and, for a loss of its own that gathers two words
// an entry, than streaming up to kVec1SmallLoss entries by one block (10K
// entries 7.6 us, 16K 9.9; with the combine 7.2 and 7.4).  Above, 256 threads of
// two entries while that does not give every SIMD two waves, of eight (16-byte
// loads) from there on.  Those are complete in one launch too, up to kVec1Whole
// entries, where no loss rides on the combine and every segment is short (SpMV
// of 262K rows of about one entry 6.6 -> 4.8 us; of 20M entries 115 -> 123).
constexpr int64_t kVec1Small = 16384;
constexpr int64_t kVec1SmallLoss = 8192;
constexpr int64_t kVec1Tail = 4096;
constexpr int64_t kVec1Whole = int64_t(1) << 23;
constexpr int32_t kVec1ShortItems = 256;
constexpr int kVec1SmallThreads = 512;
constexpr int64_t kVec1Short = int64_t(1) << 20;

static int64_t vec1_tile(int64_t nnz) {
    if (nnz <= kVec1Small) return kVec1SmallThreads;
    return kBlock * (nnz < kVec1Short ? 2 : 8);
}

// The most tiles of a pass over up to nnz entries.
int64_t vec1_max_tiles(int64_t nnz) {
    const int64_t n = std::max<int64_t>(nnz, 1), few = std::min(n, kVec1Short - 1);
    return std::max(ceil_div(n, vec1_tile(n)), ceil_div(few, vec1_tile(few)));
}

template <int T, int E, bool DUAL, bool WHOLE>
static nsd_status vec1_launch(const Vec1Params &f, int probe_id, hipStream_t st) {
    const int64_t grid = f.s.item_blocks + ceil_div(f.s.plan.nempty, T) + (f.loss ? 1 : 0);
    probe_begin(probe_id, st);
    vec1_kernel<T, E, DUAL, WHOLE><<<(unsigned)grid, T, 0, st>>>(f);
    probe_end(probe_id, st);
    return check_launch("vec1_kernel");
}

template <bool DUAL>
static nsd_status vec1_run(Vec1Params f, int probe_id, LossJob job, hipStream_t st) {
    SgrParams &a = f.s;
    const int64_t tile = vec1_tile(a.nnz);
    const int64_t tiles = ceil_div(a.nnz, tile);
    a.item_blocks = (int32_t)tiles;
    const int64_t longest = (int64_t)a.plan.longest_chunks * a.plan.item_len;
    const int64_t small = job.loss && a.X ? kVec1SmallLoss : kVec1Small;
    if (a.nnz <= small && longest <= (a.X ? 1 : 2) * kVec1Tail && !job.p1) {
        f.loss = job.loss;
        return vec1_launch<kVec1SmallThreads, 1, DUAL, true>(f, probe_id, st);
    }
    if (!job.loss && a.nnz < kVec1Whole && a.plan.nlong == 0 && a.plan.item_len <= kVec1ShortItems)
        return tile == 8 * kBlock ? vec1_launch<kBlock, 8, DUAL, true>(f, probe_id, st)
                                  : vec1_launch<kBlock, 2, DUAL, true>(f, probe_id, st);
    f.head = a.part;
    f.tail = a.part + tiles;
    if (job.loss && !job.p1) {  // the pass's own loss
        job.p1 = f.loss_part;
        job.n1 = tiles;
    }
    if (tile == 8 * kBlock) NSD_TRY((vec1_launch<kBlock, 8, DUAL, false>(f, probe_id, st)));
    else NSD_TRY((vec1_launch<kBlock, 2, DUAL, false>(f, probe_id, st)));
    probe_begin(NSD_KERNEL_SGR_FIX, st);
    vec1_fix_kernel<<<(unsigned)(ceil_div(tiles - 1, kBlockWaves) + (job.loss ? 1 : 0)), kBlock, 0,
                      st>>>(f, tile, job);
    probe_end(NSD_KERNEL_SGR_FIX, st);
    return check_launch("vec1_fix_kernel");
}

nsd_status vec1_reduce(const SgrParams &a, LossJob job, hipStream_t st) {
    Vec1Params f;
    f.s = a;
    return vec1_run<false>(f, NSD_KERNEL_SGR_MAIN, job, st);
}

nsd_status vec1_dual(const DualPass &m, const SddmmParams &entries, double *loss_part,
                     int probe_id, LossJob job, hipStream_t st) {
    Vec1Params f;
    f.s = m.s;
    f.own = m.own;
    f.sdd = m.sdd;
    f.sdd_alpha = m.sdd_alpha;
    f.entries = entries;
    if (m.count_loss) f.loss_part = loss_part;
    return vec1_run<true>(f, probe_id, job, st);
}

// ----------------------------------------------------------------- SDDMM

// out[p] = alpha X[rowidx[p]] Y[colind[p]] (X NULL: ones), entry by entry,
// with the loss beta sum w_p X Y per block.
__global__ __launch_bounds__(kBlock) void vec1_sddmm_kernel(SddmmParams a) {
    constexpr int E = kVec1SddmmEntries;
    const int64_t p0 = ((int64_t)blockIdx.x * kBlock + threadIdx.x) * E;
    double lsum = 0.0;
    if (p0 + E <= a.nnz) {
        int r[E], c[E];
        float w[E], d[E];
        load_words<E>(a.colind + p0, c);
        if (a.X) load_words<E>(a.rowidx + p0, r);
        if (a.w) load_words<E>(a.w + p0, w);
#pragma unroll
        for (int u = 0; u < E; ++u) {
            d[u] = a.Y[c[u]];
            if (a.X) d[u] *= a.X[r[u]];
        }
#pragma unroll
        for (int u = 0; u < E; ++u) {
            if (a.w) lsum += (double)w[u] * (double)d[u];
            d[u] *= a.alpha;
        }
        if (a.operm) {
            int o[E];
            load_words<E>(a.operm + p0, o);
#pragma unroll
            for (int u = 0; u < E; ++u) a.out[o[u]] = d[u];
        } else {
            store_words<E>(a.out + p0, d);
        }
    } else {
        for (int64_t p = p0; p < a.nnz; ++p) {
            const float d = a.Y[a.colind[p]] * (a.X ? a.X[a.rowidx[p]] : 1.f);
            if (a.w) lsum += (double)a.w[p] * (double)d;
            a.out[a.operm ? a.operm[p] : p] = a.alpha * d;
        }
    }
    if (a.part) {
        const double t = block_total<kBlockWaves>(lsum);
        if (threadIdx.x == 0) a.part[blockIdx.x] = a.beta * t;
    }
}

nsd_status vec1_sddmm(const SddmmParams &a, int64_t nblocks, hipStream_t st) {
    probe_begin(NSD_KERNEL_SDDMM, st);
    vec1_sddmm_kernel<<<(unsigned)nblocks, kBlock, 0, st>>>(a);
    probe_end(NSD_KERNEL_SDDMM, st);
    return check_launch("vec1_sddmm_kernel");
}

}  // namespace nsd
