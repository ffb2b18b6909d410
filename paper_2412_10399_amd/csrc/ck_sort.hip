// Cell keys, grid-block activation and the bucketing half of the particle sort.
//
// The particles are sorted stably by key = (4^3-cell block) * 64 + (cell in block),
// the G- cell being floor((x - origin)/dx + 1/4) per axis.  A stable sort by key is
// the same as a sort by (key, index), which we build in two exact stages:
//   1. bucket by block: whoever writes a particle's key (the previous G2P, or the pass
//      over the positions below) counts it into its block; the compaction enumerates
//      the blocks holding particles in increasing virtual id and, from a prefix sum of
//      the counts, gives each its range of sorted positions; every particle then takes a
//      slot in its block's fixed-size bucket with one atomic per run of particles;
//   2. inside each block (in the P2G workgroup, in LDS): order by (cell, index).
// Atomics only decide where a particle waits inside its bucket, never its final
// position, so the resulting permutation is deterministic and exact.
#include "ck_common.hpp"

#include <algorithm>

namespace ck {

namespace {

__device__ __forceinline__ int wave_lane() { return __lane_id(); }

// kMark: marks in place of block counts, written with the neighbourhood's stamps by the
// first lane of every run of equal blocks.  Particles in creation order come in short runs
// (four cells of a row): one atomic per run and stamps run by run made the pass over 4.2M
// particles 147 us (254 before the XCD order below) against 61; one scan of the bucket
// sizes afterwards takes 8.  The multi-job form counts: its jobs' other launches
// are shared with jobs that have counts.
template <bool kMark>
__device__ __forceinline__ void b_flag_keys(const DevCtx &d, const PartArgs &pa, int epoch_offset) {
    // each XCD (workgroups go to the 8 of them round-robin by index) takes a contiguous
    // eighth of the particles: rows of cells that count into the same blocks then meet in
    // one L2 (75 -> 61 us at 4.2M particles)
    const int per = (int)(gridDim.x + 7) >> 3;
    const int b = (int)(blockIdx.x & 7) * per + (int)(blockIdx.x >> 3);
    const int i = b * kThreads + (int)threadIdx.x;
    const int epoch = (int)d.counters[C_EPOCH] + epoch_offset;
    bool ok = i < pa.n;
    CellCoord cc = {};
    if (ok) {
        const float x[3] = {pa.in[i], pa.in[pa.stride + i], pa.in[2 * pa.stride + i]};
        const float xr[3] = {pa.in[kPlaneR * pa.stride + i], pa.in[(kPlaneR + 1) * pa.stride + i],
                             pa.in[(kPlaneR + 2) * pa.stride + i]};
        ok = cell_coord(d.geo, x, xr, cc);
        if (!ok) {
            d.key[i] = 0xffffffffu;
            set_status(d.counters, ST_DOMAIN);
        }
    }
    if (ok) {
        d.key[i] = cell_key(d.geo, cc);
        d.sub[i] = (uint16_t)sub_code(cc);
    }
    // every lane takes part
    const int bx = cc.c[0] >> 2, by = cc.c[1] >> 2, bz = cc.c[2] >> 2;
    if (!kMark) {
        wave_stamp(d, ok, bx, by, bz, epoch);
        return;
    }
    const Geometry &g = d.geo;
    const int vb = ok ? vblock_id(g, bx, by, bz) : -1;
    const int prev = __shfl_up(vb, 1);
    if (!ok || ((threadIdx.x & 63) != 0 && prev == vb)) return;
    block_counts(d, epoch)[vb] = 1;
    for (int z = max(bz - 1, 0); z <= min(bz + 1, g.NB[2] - 1); ++z)
        for (int y = max(by - 1, 0); y <= min(by + 1, g.NB[1] - 1); ++y)
            for (int x = max(bx - 1, 0); x <= min(bx + 1, g.NB[0] - 1); ++x) d.gflag[vblock_id(g, x, y, z)] = epoch;
}

__global__ void __launch_bounds__(kThreads) k_flag_keys(DevCtx d, PartArgs pa, int epoch_offset) {
    b_flag_keys<true>(d, pa, epoch_offset);
}

// one launch for many jobs: workgroup row y runs job y
__global__ void __launch_bounds__(kThreads) k_flag_keys_multi(const JobStep *__restrict__ jobs) {
    const JobStep &J = jobs[blockIdx.y];
    if (!J.first) return;
    b_flag_keys<false>(J.d, J.pa, 1);
}

// Ranges of sorted positions from the bucket sizes, where the blocks were only marked
// (one workgroup).
__global__ void __launch_bounds__(1024) k_bucket_scan(DevCtx d) {
    __shared__ int sh[1024 / 64];
    const int np = (int)d.counters[C_NPB];
    const int per = (np + 1023) / 1024;
    const int beg = min(np, (int)threadIdx.x * per), end = min(np, beg + per);
    int sum = 0, mx = 0;
#pragma unroll 8
    for (int i = beg; i < end; ++i) {
        const int c = d.bcount[i];
        sum += c;
        mx = max(mx, c);
    }
    if (mx > kMaxBlockParticles) set_status(d.counters, ST_CAPACITY);
    int v = sum;
    const int lane = wave_lane(), w = threadIdx.x >> 6;
#pragma unroll
    for (int off = 1; off < 64; off <<= 1) {
        const int t = __shfl_up(v, off);
        if (lane >= off) v += t;
    }
    if (lane == 63) sh[w] = v;
    __syncthreads();
    int run = v - sum;
    for (int k = 0; k < w; ++k) run += sh[k];
    for (int i = beg; i < end; ++i) {
        d.pstart[i] = run;
        run += d.bcount[i];
    }
    if (threadIdx.x == 1023) d.pstart[np] = run;
}

// The stamps go too: the last G2P made those of the epoch that is about to be sorted, for the
// particles it wrote.
__global__ void k_clear_counts(DevCtx d) {
    const long long n = 2 * stamp_stride(d.nbv) / 4;
    int4 *c = reinterpret_cast<int4 *>(d.pflag), *g = reinterpret_cast<int4 *>(d.gflag);
    for (long long v = blockIdx.x * (long long)blockDim.x + threadIdx.x; v < n; v += (long long)gridDim.x * blockDim.x) {
        c[v] = make_int4(0, 0, 0, 0);
        if (v < n / 2) g[v] = make_int4(0, 0, 0, 0);
    }
    if (one_sort(d))
        for (int r = blockIdx.x * blockDim.x + threadIdx.x; r < d.max_blocks; r += gridDim.x * blockDim.x) clear_block_record(d, r);
}

__global__ void k_reset(DevCtx d) {
    const long long t0 = blockIdx.x * (long long)blockDim.x + threadIdx.x, step = (long long)gridDim.x * blockDim.x;
    const long long nst = 2 * stamp_stride(d.nbv);
    for (long long v = t0; v < nst; v += step) {
        d.pflag[v] = 0;
        if (v < nst / 2) d.gflag[v] = 0;
        if (v < d.nbv) {
            d.page[0][v] = -1;
            d.page[1][v] = -1;
            d.prank[v] = -1;
            d.bchg[v] = -1;
        }
    }
    for (long long k = t0; k <= d.max_blocks; k += step) {
        d.pstart[k] = 0;
        if (k < d.max_blocks) clear_block_record(d, (int)k);
    }
    for (long long k = t0; k < kBoundWords; k += step) d.bslots[k] = 0u;
    if (t0 < C_COUNT) d.counters[t0] = 0u;
}

// The counters to `out` (pinned host memory: the caller waits for the stream alone, 38 us
// against 23 with a copy after the wait), with the largest particle count of a block (the
// other entries are formed by the steps).  One workgroup.
__global__ void __launch_bounds__(1024) k_stats(DevCtx d, unsigned int *out) {
    __shared__ int m;
    if (threadIdx.x == 0) m = 0;
    __syncthreads();
    const int np = (int)d.counters[C_NPB];
    int mx = 0;
    for (int r = threadIdx.x; r < np; r += 1024) mx = max(mx, d.pstart[r + 1] - d.pstart[r]);
    atomicMax(&m, mx);
    __syncthreads();
    if (threadIdx.x < C_COUNT) out[threadIdx.x] = threadIdx.x == C_MAXPB ? (unsigned)m : d.counters[threadIdx.x];
}

// Workgroup-wide sums of three counters (256 threads).
__device__ __forceinline__ void wg_sum3(int (&a)[3], int *sh) {
#pragma unroll
    for (int off = 32; off > 0; off >>= 1)
#pragma unroll
        for (int k = 0; k < 3; ++k) a[k] += __shfl_xor(a[k], off);
    const int w = threadIdx.x >> 6;
    if (wave_lane() == 0)
#pragma unroll
        for (int k = 0; k < 3; ++k) sh[3 * w + k] = a[k];
    __syncthreads();
#pragma unroll
    for (int k = 0; k < 3; ++k) {
        a[k] = 0;
#pragma unroll
        for (int q = 0; q < kThreads / 64; ++q) a[k] += sh[3 * q + k];
    }
    __syncthreads();
}

constexpr int kPerThread = kCompactChunk / kThreads;   // 4 virtual blocks per thread
// For sorts of a state that no G2P of the context wrote, and grouped jobs: chunks of 1,024
// blocks up to which one launch does the compaction, every workgroup counting the chunks
// before its own itself; for every sort on larger lattices those up to which each emitting
// workgroup sums the counts of the chunks before its own; above that a scan of the counts
// stands between.
// One launch takes 3.5 us at 5 chunks against 3.4 + 3.3 for two, but 10.2 us at 36 chunks
// against 4.7 + 4.8.  A step of 1,000 particles with sums / with the lone workgroup of a
// scan: 34.7 / 38.5 us at 892 chunks, 45.6 / 52.0 at 4,076, 60.6 / 66.0 at 7,021, 123.6 /
// 135.4 at 16,577, 318 / 307 at 32,301 and 927 / 573 at 62,970 (the sums' work grows with
// the square).
constexpr int kSingleChunks = 12;
constexpr int kPrefixChunks = 24576;

// Particle counts and grid flags (stamp == E) of the kPerThread consecutive virtual blocks
// from `base`, each array in one 16-byte load (both arrays are 256-byte aligned and padded
// to a multiple of 64 entries; entries past the last block are never counted or stamped).
__device__ __forceinline__ void load_flags(const DevCtx &d, const int *pc, long long base, int E, int (&fn)[kPerThread],
                                           int (&fg)[kPerThread]) {
    static_assert(kPerThread == 4, "one int4 per array");
    int4 a = make_int4(0, 0, 0, 0), b = make_int4(0, 0, 0, 0);
    if (base < stamp_stride(d.nbv)) {
        a = *reinterpret_cast<const int4 *>(pc + base);
        b = *reinterpret_cast<const int4 *>(d.gflag + base);
    }
    fn[0] = a.x;
    fn[1] = a.y;
    fn[2] = a.z;
    fn[3] = a.w;
    fg[0] = b.x == E;
    fg[1] = b.y == E;
    fg[2] = b.z == E;
    fg[3] = b.w == E;
}

__device__ __forceinline__ void add_flags(const int (&fn)[kPerThread], const int (&fg)[kPerThread], int (&c)[3]) {
#pragma unroll
    for (int k = 0; k < kPerThread; ++k) {
        c[0] += fn[k] != 0;
        c[1] += fg[k];
        c[2] += fn[k];
    }
}

__device__ __forceinline__ void b_compact_count(const DevCtx &d) {
    __shared__ int sh[3 * (kThreads / 64)];
    const int E = (int)d.counters[C_EPOCH] + 1;
    const long long base = (long long)blockIdx.x * kCompactChunk + threadIdx.x * kPerThread;
    int fn[kPerThread], fg[kPerThread], c[3] = {0, 0, 0};
    load_flags(d, block_counts(d, E), base, E, fn, fg);
    add_flags(fn, fg, c);
    wg_sum3(c, sh);
    if (threadIdx.x == 0) {
        d.chunk_p[blockIdx.x] = c[0];
        d.chunk_g[blockIdx.x] = c[1];
        d.chunk_n[blockIdx.x] = c[2];
    }
}

__global__ void __launch_bounds__(kThreads) k_compact_count(DevCtx d) { b_compact_count(d); }

__device__ __forceinline__ int chunk_count(const DevCtx &d) { return (int)((d.nbv + kCompactChunk - 1) / kCompactChunk); }

// one launch for many jobs: workgroup row y runs job y
__global__ void __launch_bounds__(kThreads) k_compact_count_multi(const JobStep *__restrict__ jobs) {
    const JobStep &J = jobs[blockIdx.y];
    if ((int)blockIdx.x >= chunk_count(J.d)) return;
    b_compact_count(J.d);
}

// Exclusive scan of an array of `n` ints in place by one workgroup of T threads.
template <int T>
__device__ void wg_scan_inplace(int *da, int n, int *sh) {
    const int per = (n + T - 1) / T;
    const int beg = min(n, (int)threadIdx.x * per), end = min(n, beg + per);
    int la = 0;
    for (int i = beg; i < end; ++i) la += da[i];
    // inclusive scan of the per-thread sums across the workgroup
    int va = la;
    const int lane = wave_lane();
#pragma unroll
    for (int off = 1; off < 64; off <<= 1) {
        const int t = __shfl_up(va, off);
        if (lane >= off) va += t;
    }
    const int w = threadIdx.x >> 6;
    if (lane == 63) sh[w] = va;
    __syncthreads();
    int pre = 0;
    for (int k = 0; k < w; ++k) pre += sh[k];
    int ra = pre + va - la;
    for (int i = beg; i < end; ++i) {
        const int t = da[i];
        da[i] = ra;
        ra += t;
    }
    __syncthreads();
}

__device__ __forceinline__ void b_compact_scan(const DevCtx &d, int nchunks) {
    __shared__ int sh[1024 / 64];
    wg_scan_inplace<1024>(d.chunk_p, nchunks, sh);
    wg_scan_inplace<1024>(d.chunk_g, nchunks, sh);
    wg_scan_inplace<1024>(d.chunk_n, nchunks, sh);
}

__global__ void __launch_bounds__(1024) k_compact_scan(DevCtx d, int nchunks) { b_compact_scan(d, nchunks); }

// one launch for many jobs: workgroup row y runs job y
__global__ void __launch_bounds__(1024) k_compact_scan_multi(const JobStep *__restrict__ jobs) {
    const JobStep &J = jobs[blockIdx.y];
    b_compact_scan(J.d, chunk_count(J.d));
}

// Workgroup exclusive scan of three ints per thread (256 threads).
__device__ __forceinline__ void wg_excl_scan3(const int (&x)[3], int (&excl)[3], int *sh) {
    int v[3] = {x[0], x[1], x[2]};
    const int lane = wave_lane();
#pragma unroll
    for (int off = 1; off < 64; off <<= 1)
#pragma unroll
        for (int q = 0; q < 3; ++q) {
            const int t = __shfl_up(v[q], off);
            if (lane >= off) v[q] += t;
        }
    const int w = threadIdx.x >> 6;
    if (lane == 63)
#pragma unroll
        for (int q = 0; q < 3; ++q) sh[3 * w + q] = v[q];
    __syncthreads();
#pragma unroll
    for (int q = 0; q < 3; ++q) {
        int pre = 0;
#pragma unroll
        for (int k = 0; k < kThreads / 64; ++k) pre += (k < w) ? sh[3 * k + q] : 0;
        excl[q] = pre + v[q] - x[q];
    }
}

// Page table entries, block lists, and the particle blocks' ranges of sorted positions of
// kPerThread virtual blocks from `base`, whose particle blocks, grid blocks and particles
// start at first[]; `last`: the thread of the last virtual blocks.  kOneLaunch: the records
// of the blocks' orders are filled by the same launch and were cleared before it.
template <bool kOneLaunch>
__device__ __forceinline__ void emit_blocks(const DevCtx &d, int table, int E, long long base, const int (&fn)[kPerThread],
                                            const int (&fg)[kPerThread], const int (&first)[3], bool last) {
    int rp = first[0], rg = first[1], rn = first[2];
    if (last) {
        int c[3] = {0, 0, 0};
        add_flags(fn, fg, c);
        const int np = rp + c[0], ng = rg + c[1];
        if (ng > d.max_blocks || np > d.max_blocks) set_status(d.counters, ST_CAPACITY);
        d.counters[C_NPB] = (unsigned)min(np, d.max_blocks);
        d.counters[ngb_slot(table)] = (unsigned)min(ng, d.max_blocks);
        d.counters[C_SORT] = (unsigned)E;
        if (np <= d.max_blocks) d.pstart[np] = rn + c[2];
    }
    int ph[kPerThread];
#pragma unroll
    for (int k = 0; k < kPerThread; ++k) {
        const int v = (int)(base + k);
        if (fn[k]) {
            if (rp < d.max_blocks) {
                d.plist[rp] = v;
                d.prank[v] = rp;
                d.pstart[rp] = rn;
                if (!kOneLaunch) clear_block_record(d, rp);
                if (fn[k] > kMaxBlockParticles) set_status(d.counters, ST_CAPACITY);
            } else {
                if (rp == d.max_blocks) d.pstart[rp] = rn;
                d.prank[v] = -1;
            }
            ++rp;
            rn += fn[k];
        }
        ph[k] = -1;
        if (fg[k]) {
            if (rg < d.max_blocks) {
                glist_of(d, table)[rg] = v;
                ph[k] = rg;
            }
            ++rg;
        }
    }
    // every virtual block gets its page entry, so the table is valid without stamps
    if (base + kPerThread <= d.nbv) {
        *reinterpret_cast<int4 *>(page_of(d, table) + base) = make_int4(ph[0], ph[1], ph[2], ph[3]);
    } else {
#pragma unroll
        for (int k = 0; k < kPerThread; ++k)
            if (base + k < d.nbv) page_of(d, table)[base + k] = ph[k];
    }
}

// How the emission learns what the chunks before its own hold.
enum EmitFrom {
    EMIT_FLAGS = 0,    // counts them itself from the counts and stamps (no other launch)
    EMIT_COUNTS = 1,   // sums the chunk counts before its own
    EMIT_SCAN = 2      // the chunk counts have been scanned
};

// Page table entries, block lists, and the particle blocks' ranges of sorted positions
// for one chunk of virtual blocks.
template <int kFrom>
__device__ __forceinline__ void b_compact_emit(const DevCtx &d, int table, int nchunks) {
    __shared__ int sh[3 * (kThreads / 64)], sh2[3 * (kThreads / 64)];
    const int E = (int)d.counters[C_EPOCH] + 1;
    const int *pc = block_counts(d, E);
    const long long base = (long long)blockIdx.x * kCompactChunk + threadIdx.x * kPerThread;
    int fn[kPerThread], fg[kPerThread], c[3] = {0, 0, 0}, before[3] = {0, 0, 0}, ex[3];
    load_flags(d, pc, base, E, fn, fg);
    if (kFrom == EMIT_FLAGS) {
#pragma unroll 4
        for (int q = 0; q < (int)blockIdx.x; ++q) {
            int an[kPerThread], ag[kPerThread];
            load_flags(d, pc, (long long)q * kCompactChunk + threadIdx.x * kPerThread, E, an, ag);
            add_flags(an, ag, before);
        }
        wg_sum3(before, sh2);
    } else if (kFrom == EMIT_COUNTS) {
        for (int q = threadIdx.x; q < (int)blockIdx.x; q += kThreads) {
            before[0] += d.chunk_p[q];
            before[1] += d.chunk_g[q];
            before[2] += d.chunk_n[q];
        }
        wg_sum3(before, sh2);
    } else {
        before[0] = d.chunk_p[blockIdx.x];
        before[1] = d.chunk_g[blockIdx.x];
        before[2] = d.chunk_n[blockIdx.x];
    }
    add_flags(fn, fg, c);
    wg_excl_scan3(c, ex, sh);
    const int first[3] = {before[0] + ex[0], before[1] + ex[1], before[2] + ex[2]};
    emit_blocks<false>(d, table, E, base, fn, fg, first, (int)blockIdx.x == nchunks - 1 && threadIdx.x == kThreads - 1);
}

template <int kFrom>
__global__ void __launch_bounds__(kThreads) k_compact_emit(DevCtx d, int table, int nchunks) {
    b_compact_emit<kFrom>(d, table, nchunks);
}

// one launch for many jobs: workgroup row y runs job y
template <int kFrom>
__global__ void __launch_bounds__(kThreads) k_compact_emit_multi(const JobStep *__restrict__ jobs) {
    const JobStep &J = jobs[blockIdx.y];
    const int nchunks = chunk_count(J.d);
    if ((int)blockIdx.x >= nchunks) return;
    b_compact_emit<kFrom>(J.d, J.table, nchunks);
}

// Each particle takes a slot in its block's bucket and writes its index there.
// Particles arrive nearly sorted (the previous G2P wrote them in block order), so
// a workgroup's 1024 consecutive particles span few blocks: slots are ranked
// inside the workgroup (a run of equal blocks gets consecutive slots) and each run
// costs one global atomic.  Slots past the bucket capacity are not written (the
// compaction reports such a block).  The same launch zeroes this step's grid blocks,
// makes the sort's epoch the current one and reduces the P2G contribution bound.
constexpr int kCountPer = 4;                       // consecutive particles per thread
constexpr int kCountTile = kThreads * kCountPer;   // particles per workgroup

// By the first workgroup of a sort's last launch: the contribution bound for the P2G about
// to run is formed from the maxima of the slots the previous P2G (or the stress pass)
// filled, which are cleared for the next.  Empty slots (a sequence of fused steps, which
// form no bound) leave the last bound in place.
__device__ __forceinline__ void bound_of_slots(const DevCtx &d) {
    static_assert(kBoundSlots == 64, "one wave reduces the slots");
    const int tid = threadIdx.x;
    if (tid < kBoundSlots) {
        unsigned int *sx = d.bslots + tid * 32, *sy = d.bslots + (kBoundSlots + tid) * 32;
        unsigned int bxv = *sx, byv = *sy;
        *sx = 0u;
        *sy = 0u;
#pragma unroll
        for (int off = 32; off > 0; off >>= 1) {
            bxv = max(bxv, (unsigned int)__shfl_xor((int)bxv, off));
            byv = max(byv, (unsigned int)__shfl_xor((int)byv, off));
        }
        if (tid == 0 && (bxv | byv) != 0u) {
            d.counters[C_BOUND_X] = bxv;
            d.counters[C_BOUND_Y] = byv;
        }
    }
}

// Start of the run of equal blocks each of a thread's particles belongs to, from the
// tile's blocks vblk: inclusive max-scan of (element starts a run ? position : 0), here
// within the thread (returns its maximum) ...
__device__ __forceinline__ int run_starts(const uint32_t *vblk, const uint32_t (&vb)[kCountPer], int (&st)[kCountPer]) {
    int m = 0;
#pragma unroll
    for (int k = 0; k < kCountPer; ++k) {
        const int j = (int)threadIdx.x * kCountPer + k;
        const bool starts = (j == 0) || (vblk[j - 1] != vb[k]);
        m = starts ? j : m;
        st[k] = m;
    }
    return m;
}
// ... and over the threads before: v the wave's inclusive maxima, wmax every wave's.
__device__ __forceinline__ void finish_runs(const int *wmax, int v, int (&st)[kCountPer]) {
    const int lane = wave_lane(), w = threadIdx.x >> 6;
    int carry = 0;
    for (int k = 0; k < w; ++k) carry = max(carry, wmax[k]);
    const int up = __shfl_up(v, 1);                       // every lane takes part in the shuffle
    const int prev_thread = lane > 0 ? max(carry, up) : carry;   // max over all earlier threads
#pragma unroll
    for (int k = 0; k < kCountPer; ++k) st[k] = max(st[k], prev_thread);
}

// reuse: the state is the one the context's previous G2P wrote; a block that G2P
// left unchanged keeps its order in the P2G (its particles sit at consecutive
// positions), so its bucket is not filled: the run's first and last positions go to
// the block's position range instead.
__device__ __forceinline__ void b_bucket_count(const DevCtx &d, int n, int zero_pool, int zero_table, bool reuse) {
    constexpr uint32_t kNone = 0xffffffffu >> 6;   // block of a particle that is not placed
    __shared__ uint32_t vblk[kCountTile];   // virtual block of each particle of the tile
    __shared__ int rank_of[kCountTile];     // per run start: particle block, -1 when nothing is written
    __shared__ int base_of[kCountTile];     // and the run's first slot
    __shared__ int wmax[kThreads / 64];
    const int tid = threadIdx.x, lane = wave_lane(), w = tid >> 6;
    const int E = (int)d.counters[C_SORT];   // the epoch of this sort
    int *pc = block_counts(d, E);
    // the tile in launch order: with a contiguous eighth for each XCD, rows of a state in creation
    // order met at their blocks' counters at once (32.2 us against 23.3 at 300,000 particles,
    // 38.7 / 31.9 at 1,000,000, 107 / 113 at 4,200,000; a state in block order takes the same)
    const int base = (int)blockIdx.x < (n + kCountTile - 1) / kCountTile ? (int)blockIdx.x * kCountTile : n;
    const int i0 = base + tid * kCountPer;
    uint32_t vb[kCountPer];
    // the thread's 4 keys in one 16-byte load (the library's buffers are 256-byte
    // aligned), element loads at the tail
    static_assert(kCountPer == 4, "vector loads take 4 keys");
    if (i0 + kCountPer <= n) {
        const uint4 k4 = *reinterpret_cast<const uint4 *>(d.key + i0);
        vb[0] = k4.x >> 6;
        vb[1] = k4.y >> 6;
        vb[2] = k4.z >> 6;
        vb[3] = k4.w >> 6;
    } else {
#pragma unroll
        for (int k = 0; k < kCountPer; ++k) vb[k] = i0 + k < n ? d.key[i0 + k] >> 6 : kNone;
    }
    // the sort's epoch becomes the current one (the other workgroups do not read it)
    if (blockIdx.x == 0) {
        bound_of_slots(d);
        if (tid == 0) d.counters[C_EPOCH] = (unsigned)E;
    }
    // zero a share of the pool blocks handed out this step
    {
        const long long nfl = (long long)d.counters[ngb_slot(zero_table)] * (kBlockFloats / 4);
        float4 *pool4 = reinterpret_cast<float4 *>(pool_of(d, zero_pool));
        for (long long t = (long long)blockIdx.x * kThreads + tid; t < nfl; t += (long long)gridDim.x * kThreads)
            pool4[t] = make_float4(0.0f, 0.0f, 0.0f, 0.0f);
    }
    if (base >= n) return;   // the whole workgroup: pool blocks only
#pragma unroll
    for (int k = 0; k < kCountPer; ++k) vblk[tid * kCountPer + k] = vb[k];
    lds_barrier();
    int st[kCountPer];
    const int v = wave_maxima(run_starts(vblk, vb, st));
    if (lane == 63) wmax[w] = v;
    lds_barrier();
    finish_runs(wmax, v, st);
    // the last element of each run looks its block up and takes the run's slots with one
    // atomic
#pragma unroll
    for (int k = 0; k < kCountPer; ++k) {
        const int j = tid * kCountPer + k;
        const bool last = (j == kCountTile - 1) || (vblk[j + 1] != vb[k]);
        if (!last) continue;
        int r = -1;
        if (vb[k] != kNone) {
            // a key whose block counts no particles this step cannot be placed
            const int f = pc[vb[k]], pr = d.prank[vb[k]], chg = d.bchg[vb[k]];
            if (f == 0) {
                set_status(d.counters, ST_STALE);
            } else if (pr < 0) {
                pc[vb[k]] = 0;   // past the capacity: no G2P visits this block
            } else if (reuse && chg != E) {
                atomicMin(&d.blo[pr], (uint32_t)(base + st[k]));
                atomicMax(&d.bhi[pr], (uint32_t)(base + j));
            } else {
                r = pr;
                base_of[st[k]] = atomicAdd(&d.bcount[pr], j - st[k] + 1);
            }
        }
        rank_of[st[k]] = r;
    }
    lds_barrier();
#pragma unroll
    for (int k = 0; k < kCountPer; ++k) {
        const int j = tid * kCountPer + k;
        const int r = rank_of[st[k]];
        if (r < 0) continue;
        const int slot = base_of[st[k]] + (j - st[k]);
        if (slot < kMaxBlockParticles) {
            d.bucket[(size_t)r * kMaxBlockParticles + slot] = (uint32_t)(base + j);
            d.bsub[(size_t)r * kMaxBlockParticles + slot] = d.sub[base + j];
        }
    }
}

// The whole sort of a state that the context's previous G2P wrote, in one launch, for
// lattices of up to kOneSortChunks chunks: every workgroup forms the ranks of all particle
// blocks itself (LDS, from the counts), so that its particles need no table from another
// launch; the first workgroups write the tables that later launches read, one chunk each.
// Nothing that the launch reads is written by it: the epoch it starts from stays current
// until P2G, and the records of the blocks' orders were cleared by the last reader (P2G).
// Bound by latency: three dependent round trips.  Measured
// against the separate compaction and bucketing: 6.2 us for 3.6 + 5.6 at 1,000 particles
// (1 chunk), 6.6 us for 4.7 + 7.6 at 32,768; a whole step 30.6 -> 26.5 us and 43.1 -> 38.4 us.
__device__ __forceinline__ void b_sort_once(const DevCtx &d, int n, int table, int nchunks) {
    constexpr uint32_t kNone = 0xffffffffu >> 6;
    constexpr int kWaves = kThreads / 64, kRanges = kOneSortChunks * kWaves;
    static_assert(kRanges <= 64 && kCountPer == 4 && kPerThread == 4, "one wave scans the ranges");
    __shared__ uint16_t blocks[kOneSortChunks * kThreads];   // per 4 virtual blocks: rank in its wave's 256, flags << 12
    __shared__ int part[3][kRanges + 1];                     // per wave's range: particle blocks, grid blocks, particles
    __shared__ uint32_t vblk[kCountTile];
    __shared__ int rank_of[kCountTile];
    __shared__ int base_of[kCountTile];
    __shared__ int wmax[kWaves];
    const int tid = threadIdx.x, lane = wave_lane(), w = tid >> 6;
    const int E = (int)d.counters[C_EPOCH] + 1;
    const int tiles = (n + kCountTile - 1) / kCountTile, per = (tiles + 7) >> 3;
    const int tile = (int)(blockIdx.x >> 3) < per ? (int)(blockIdx.x & 7) * per + (int)(blockIdx.x >> 3) : -1;
    const int base = tile >= 0 && tile < tiles ? tile * kCountTile : n;
    const int i0 = base + tid * kCountPer;
    uint32_t vb[kCountPer];
    uint32_t sub[kCountPer];
    if (i0 + kCountPer <= n) {
        const uint4 k4 = *reinterpret_cast<const uint4 *>(d.key + i0);
        const uint2 s4 = *reinterpret_cast<const uint2 *>(d.sub + i0);
        vb[0] = k4.x >> 6;
        vb[1] = k4.y >> 6;
        vb[2] = k4.z >> 6;
        vb[3] = k4.w >> 6;
        sub[0] = s4.x & 0xffffu;
        sub[1] = s4.x >> 16;
        sub[2] = s4.y & 0xffffu;
        sub[3] = s4.y >> 16;
    } else {
#pragma unroll
        for (int k = 0; k < kCountPer; ++k) {
            vb[k] = i0 + k < n ? d.key[i0 + k] >> 6 : kNone;
            sub[k] = i0 + k < n ? d.sub[i0 + k] : 0u;
        }
    }
    if (blockIdx.x == 0) bound_of_slots(d);
    // ranks of the particle blocks, and the share of every wave's 256 virtual blocks
    const int *pc = block_counts(d, E);
    int fn[kPerThread] = {}, fg[kPerThread] = {}, ex[3] = {};   // of this workgroup's chunk, if it writes one
    constexpr int kBatch = 4;   // chunks whose loads are in flight together
    for (int q0 = 0; q0 < nchunks; q0 += kBatch) {
        int an[kBatch][kPerThread], ag[kBatch][kPerThread];
#pragma unroll
        for (int i = 0; i < kBatch; ++i)
            if (q0 + i < nchunks) load_flags(d, pc, (long long)(q0 + i) * kCompactChunk + tid * kPerThread, E, an[i], ag[i]);
#pragma unroll
        for (int i = 0; i < kBatch; ++i) {
            const int q = q0 + i;
            if (q >= nchunks) break;
            int c[3] = {0, 0, 0};
            add_flags(an[i], ag[i], c);
            const int sum[3] = {wave_sums(c[0]), wave_sums(c[1]), wave_sums(c[2])};
            const int flags = (an[i][0] != 0) | (an[i][1] != 0) << 1 | (an[i][2] != 0) << 2 | (an[i][3] != 0) << 3;
            blocks[q * kThreads + tid] = (uint16_t)((sum[0] - c[0]) | flags << 12);
            if (lane == 63)
#pragma unroll
                for (int k = 0; k < 3; ++k) part[k][q * kWaves + w] = sum[k];
            if (q == (int)blockIdx.x) {
#pragma unroll
                for (int k = 0; k < kPerThread; ++k) {
                    fn[k] = an[i][k];
                    fg[k] = ag[i][k];
                }
#pragma unroll
                for (int k = 0; k < 3; ++k) ex[k] = sum[k] - c[k];
            }
        }
    }
    // the start of the run of equal blocks each particle belongs to, as in the bucketing
#pragma unroll
    for (int k = 0; k < kCountPer; ++k) vblk[tid * kCountPer + k] = vb[k];
    lds_barrier();
    if (w < 3) {
        const int e = lane < nchunks * kWaves ? part[w][lane] : 0;
        const int s = wave_sums(e);
        if (lane < kRanges) part[w][lane] = s - e;
        if (lane == 63) part[w][kRanges] = s;
    }
    int st[kCountPer];
    const int v = wave_maxima(run_starts(vblk, vb, st));
    if (lane == 63) wmax[w] = v;
    lds_barrier();
    // zero a share of the pool blocks handed out this step
    {
        const long long nfl = (long long)min(part[1][kRanges], d.max_blocks) * (kBlockFloats / 4);
        float4 *pool4 = reinterpret_cast<float4 *>(pool_of(d, table));
        for (long long t = (long long)blockIdx.x * kThreads + tid; t < nfl; t += (long long)gridDim.x * kThreads)
            pool4[t] = make_float4(0.0f, 0.0f, 0.0f, 0.0f);
    }
    if (base < n) {
        finish_runs(wmax, v, st);
#pragma unroll
        for (int k = 0; k < kCountPer; ++k) {
            const int j = tid * kCountPer + k;
            const bool last = (j == kCountTile - 1) || (vblk[j + 1] != vb[k]);
            if (!last) continue;
            int r = -1;
            if (vb[k] != kNone) {
                const uint32_t f = blocks[vb[k] >> 2], in = vb[k] & 3u;
                const int pr = part[0][vb[k] >> 8] + (int)(f & 0xfffu) + __popc((f >> 12) & ((1u << in) - 1u));
                if (((f >> (12 + in)) & 1u) == 0) {
                    set_status(d.counters, ST_STALE);   // no particles were counted into its block
                } else if (pr < d.max_blocks) {
                    if (d.bchg[vb[k]] != E) {
                        atomicMin(&d.blo[pr], (uint32_t)(base + st[k]));
                        atomicMax(&d.bhi[pr], (uint32_t)(base + j));
                    } else {
                        r = pr;
                        base_of[st[k]] = atomicAdd(&d.bcount[pr], j - st[k] + 1);
                    }
                }
            }
            rank_of[st[k]] = r;
        }
        lds_barrier();
#pragma unroll
        for (int k = 0; k < kCountPer; ++k) {
            const int j = tid * kCountPer + k;
            const int r = rank_of[st[k]];
            if (r < 0) continue;
            const int slot = base_of[st[k]] + (j - st[k]);
            if (slot < kMaxBlockParticles) {
                d.bucket[(size_t)r * kMaxBlockParticles + slot] = (uint32_t)(base + j);
                d.bsub[(size_t)r * kMaxBlockParticles + slot] = (uint16_t)sub[k];
            }
        }
    }
    if ((int)blockIdx.x < nchunks) {
        const int first[3] = {part[0][blockIdx.x * kWaves + w] + ex[0], part[1][blockIdx.x * kWaves + w] + ex[1],
                              part[2][blockIdx.x * kWaves + w] + ex[2]};
        emit_blocks<true>(d, table, E, (long long)blockIdx.x * kCompactChunk + tid * kPerThread, fn, fg, first,
                          (int)blockIdx.x == nchunks - 1 && tid == kThreads - 1);
    }
}

__global__ void __launch_bounds__(kThreads) k_sort_once(DevCtx d, int n, int table, int nchunks) {
    b_sort_once(d, n, table, nchunks);
}

__global__ void __launch_bounds__(kThreads) k_bucket_count(DevCtx d, int n, int zero_pool, int zero_table, int reuse) {
    b_bucket_count(d, n, zero_pool, zero_table, reuse != 0);
}

// one launch for many jobs: workgroup row y runs job y
__global__ void __launch_bounds__(kThreads) k_bucket_count_multi(const JobStep *__restrict__ jobs) {
    const JobStep &J = jobs[blockIdx.y];
    // a job's steps after its first read the state its own G2P wrote
    b_bucket_count(J.d, J.pa.n, J.table, J.table, !J.first);
}

}  // namespace

namespace {
int flag_blocks(int n) { return (n + 8 * kThreads - 1) / (8 * kThreads) * 8; }
}  // namespace

void launch_flag_keys(const DevCtx &d, const PartArgs &pa, int epoch_offset, hipStream_t s) {
    if (pa.n <= 0) return;
    hipLaunchKernelGGL(k_flag_keys, dim3(flag_blocks(pa.n)), dim3(kThreads), 0, s, d, pa, epoch_offset);
}

void launch_clear_counts(const DevCtx &d, hipStream_t s) {
    const long long wgs = (2 * stamp_stride(d.nbv) / 4 + 255) / 256;
    hipLaunchKernelGGL(k_clear_counts, dim3((unsigned)std::min<long long>(wgs, 1024)), dim3(256), 0, s, d);
}

void launch_reset(const DevCtx &d, hipStream_t s) {
    const long long wgs = std::max<long long>(2 * stamp_stride(d.nbv), std::max<long long>(d.max_blocks, kBoundWords)) / 256 + 1;
    hipLaunchKernelGGL(k_reset, dim3((unsigned)std::min<long long>(wgs, 1024)), dim3(256), 0, s, d);
}

void launch_stats(const DevCtx &d, unsigned int *out, hipStream_t s) {
    hipLaunchKernelGGL(k_stats, dim3(1), dim3(1024), 0, s, d, out);
}

void launch_compact(const DevCtx &d, int table, hipStream_t s) {
    const int nchunks = (int)((d.nbv + kCompactChunk - 1) / kCompactChunk);
    const dim3 grid(nchunks), wg(kThreads);
    if (nchunks <= kSingleChunks) {
        hipLaunchKernelGGL(k_compact_emit<EMIT_FLAGS>, grid, wg, 0, s, d, table, nchunks);
        return;
    }
    hipLaunchKernelGGL(k_compact_count, grid, wg, 0, s, d);
    if (nchunks <= kPrefixChunks) {
        hipLaunchKernelGGL(k_compact_emit<EMIT_COUNTS>, grid, wg, 0, s, d, table, nchunks);
    } else {
        hipLaunchKernelGGL(k_compact_scan, dim3(1), dim3(1024), 0, s, d, nchunks);
        hipLaunchKernelGGL(k_compact_emit<EMIT_SCAN>, grid, wg, 0, s, d, table, nchunks);
    }
}

namespace {

// Workgroups of the bucketing: one per tile of particles, and enough to spread the clearing
// of the pool (at most max_blocks blocks of 128 float4, eight float4 per thread) up to
// 1,024.
int bucket_blocks(const DevCtx &d, int n) {
    const int tiles = ((n + kCountTile - 1) / kCountTile + 7) / 8 * 8;
    const int zero = (int)std::min<long long>(1024, ((long long)d.max_blocks * (kBlockFloats / 4) + 8 * kThreads - 1) / (8 * kThreads));
    return std::max(std::max(tiles, zero), 1);
}

}  // namespace

void launch_sort_multi(const JobStep *dev, const JobStep *host, int njobs, hipStream_t s) {
    int flag_grid = 0, chunks = 1, tiles = 1;
    for (int j = 0; j < njobs; ++j) {
        const JobStep &J = host[j];
        if (J.first) flag_grid = std::max(flag_grid, flag_blocks(J.pa.n));
        chunks = std::max(chunks, (int)((J.d.nbv + kCompactChunk - 1) / kCompactChunk));
        tiles = std::max(tiles, bucket_blocks(J.d, J.pa.n));
    }
    const dim3 cg(chunks, njobs), wg(kThreads);
    if (flag_grid > 0) hipLaunchKernelGGL(k_flag_keys_multi, dim3(flag_grid, njobs), wg, 0, s, dev);
    if (chunks <= kSingleChunks) {
        hipLaunchKernelGGL(k_compact_emit_multi<EMIT_FLAGS>, cg, wg, 0, s, dev);
    } else {
        hipLaunchKernelGGL(k_compact_count_multi, cg, wg, 0, s, dev);
        if (chunks <= kPrefixChunks) {
            hipLaunchKernelGGL(k_compact_emit_multi<EMIT_COUNTS>, cg, wg, 0, s, dev);
        } else {
            hipLaunchKernelGGL(k_compact_scan_multi, dim3(1, njobs), dim3(1024), 0, s, dev);
            hipLaunchKernelGGL(k_compact_emit_multi<EMIT_SCAN>, cg, wg, 0, s, dev);
        }
    }
    hipLaunchKernelGGL(k_bucket_count_multi, dim3(tiles, njobs), wg, 0, s, dev);
}

void launch_sort_once(const DevCtx &d, int n, int table, hipStream_t s) {
    const int nchunks = (int)((d.nbv + kCompactChunk - 1) / kCompactChunk);
    hipLaunchKernelGGL(k_sort_once, dim3(std::max(bucket_blocks(d, n), nchunks)), dim3(kThreads), 0, s, d, n, table, nchunks);
}

void launch_bucket(const DevCtx &d, int n, int zero_pool, int zero_table, hipStream_t s, bool reuse, bool marked) {
    hipLaunchKernelGGL(k_bucket_count, dim3(bucket_blocks(d, n)), dim3(kThreads), 0, s, d, n, zero_pool, zero_table,
                       reuse ? 1 : 0);
    if (marked) hipLaunchKernelGGL(k_bucket_scan, dim3(1), dim3(1024), 0, s, d);
}

}  // namespace ck
