// Dispatch plan: per-expert counts, prefix sums, stable grouping of assignments by expert,
// execution order of the experts, and the tile tables the grouped FFN walks.
//
// The expert layer is evaluated expert by expert over the tokens of all batches of the batch
// group, experts that serve the most batches / tokens first (paper Section 5).  Everything
// here is integer work with a unique answer: histograms use LDS atomics (order-free), stable
// ranks come from wavefront ballots and per-segment prefix sums.
#include "kernels.h"

namespace kmoe {
namespace {

constexpr int kThreads = 256;
constexpr int kRounds = kPlanChunk / kThreads;  // 4
constexpr int kSegs = kRounds * (kThreads / 64);  // 16 (round, wave) segments per chunk

// The batch offsets arrive as a kernel argument; a per-lane index into them would be a chain of
// dependent global loads, so they are first copied to LDS (sbo, kMaxBatches + 1 ints).
__device__ __forceinline__ void stage_offsets(const BatchOffsets& bo, int32_t* sbo) {
    for (int b = threadIdx.x; b <= kMaxBatches; b += kThreads) sbo[b] = bo.v[b];
}

__device__ __forceinline__ int batch_of(const int32_t* sbo, int n, int t) {
    int lo = 0, hi = n;  // find b with v[b] <= t < v[b+1]
    while (hi - lo > 1) {
        int mid = (lo + hi) >> 1;
        if (sbo[mid] <= t) lo = mid; else hi = mid;
    }
    return lo;
}

// Lanes of the wavefront whose assignment goes to the same expert as this lane's (0 for lanes without
// one, e < 0): one ballot per bit of the expert id.
__device__ __forceinline__ unsigned long long same_expert(int e, int ebits) {
    unsigned long long m = __ballot(e >= 0);
    for (int b = 0; b < ebits; ++b) {
        const bool bit = (e >> b) & 1;
        const unsigned long long ones = __ballot(bit);
        m &= bit ? ones : ~ones;
    }
    return e >= 0 ? m : 0ull;
}
__device__ __forceinline__ int bits_for(int E) { return 32 - __clz(E - 1 > 0 ? E - 1 : 1); }  // ids 0 .. E-1
__device__ __forceinline__ unsigned long long lanes_below() { return (1ull << (threadIdx.x & 63)) - 1ull; }

// Adds batch b of assignments to expert e to the expert's batch mask.  Consecutive lanes with the
// same expert mostly come from the same batch: a lane whose predecessor in `same` does leaves the
// (serialising) LDS atomic to it.
__device__ __forceinline__ void add_batch(unsigned long long* msk, int e, int b, unsigned long long same) {
    const unsigned long long before = same & lanes_below();
    const int prev = before ? 63 - __clzll((long long)before) : (int)(threadIdx.x & 63);
    const int bp = __shfl(b, prev, 64);
    if (e >= 0 && (before == 0ull || bp != b)) atomicOr(&msk[e], 1ull << b);
}

// P1: per chunk of assignments, tokens per expert and the set of batches touching each expert.
__global__ __launch_bounds__(kThreads) void plan_count_kernel(const int32_t* __restrict__ idx,
                                                              int A, int E, int k, BatchOffsets bo,
                                                              int32_t* __restrict__ blk_counts,
                                                              unsigned long long* __restrict__ blk_mask) {
    __shared__ int32_t cnt[kMaxExperts];
    __shared__ unsigned long long msk[kMaxExperts];
    __shared__ int32_t sbo[kMaxBatches + 1];
    const int base = blockIdx.x * kPlanChunk;
    int mine[kRounds];
#pragma unroll
    for (int r = 0; r < kRounds; ++r) {
        const int a = base + r * kThreads + threadIdx.x;
        mine[r] = a < A ? idx[a] : -1;
    }
    stage_offsets(bo, sbo);
    for (int e = threadIdx.x; e < E; e += kThreads) {
        cnt[e] = 0;
        msk[e] = 0ull;
    }
    __syncthreads();
    const int ebits = bits_for(E);
#pragma unroll
    for (int r = 0; r < kRounds; ++r) {
        const int a = base + r * kThreads + threadIdx.x, e = mine[r];
        const unsigned long long same = same_expert(e, ebits);
        if (e >= 0 && (same & lanes_below()) == 0ull) atomicAdd(&cnt[e], __popcll(same));
        add_batch(msk, e, a < A ? batch_of(sbo, bo.n, a / k) : 0, same);
    }
    __syncthreads();
    for (int e = threadIdx.x; e < E; e += kThreads) {
        blk_counts[(size_t)blockIdx.x * E + e] = cnt[e];
        blk_mask[(size_t)blockIdx.x * E + e] = msk[e];
    }
}

// LDS of the scans: one entry per expert.
struct ScanLds {
    int32_t cnt[kMaxExperts];  // tokens (set by the caller)
    int32_t nbt[kMaxExperts];  // batches (set by the caller)
    int32_t off[kMaxExperts + 1], pof[kMaxExperts + 1];
    int32_t ord[kMaxExperts];
    unsigned long long key[kMaxExperts];
    int32_t wsum[2][kMaxExperts / 64];
};

// Exclusive sums over the first kMaxExperts threads of the workgroup (whole wavefronts) of two
// values at once; every thread calls it.
__device__ __forceinline__ void scan2(int& a, int& b, int& total_a, int& total_b, int32_t (*wsum)[kMaxExperts / 64]) {
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    int sa = a, sb = b;
#pragma unroll
    for (int m = 1; m < 64; m <<= 1) {
        const int ua = __shfl_up(sa, m, 64), ub = __shfl_up(sb, m, 64);
        if (lane >= m) {
            sa += ua;
            sb += ub;
        }
    }
    __syncthreads();  // wsum of an earlier call has been read
    if (lane == 63 && wave < kMaxExperts / 64) {
        wsum[0][wave] = sa;
        wsum[1][wave] = sb;
    }
    __syncthreads();
    total_a = total_b = 0;
    int before_a = 0, before_b = 0;
#pragma unroll
    for (int w = 0; w < kMaxExperts / 64; ++w) {
        if (w == wave) {
            before_a = total_a;
            before_b = total_b;
        }
        total_a += wsum[0][w];
        total_b += wsum[1][w];
    }
    a = sa - a + before_a;
    b = sb - b + before_b;
}

// First row block of tile j of an expert's n blocks (n for j = tiles).  Up to kEvenTiles tiles are cut
// evenly (they differ by one block at most), more are full tiles and a rest: an uneven last tile of few
// leaves the last workgroups of a launch uneven, among many it does not matter.  Uneven / even, 8 experts
// of 4096 x 14336, top-2: two tiles 1300 tokens 1185 / 1023 us, 1800 1309 / 1251; three 2600 1919 / 1839; four 3300
// 2260 / 2167, 3900 2417 / 2427; five to eight, between 4300 and 8100 tokens, from 2907 / 2801 (4300) to 4556 / 4660
// (7700); 16 and 17 9.92 / 10.00 ms.
constexpr int kEvenTiles = 4;
__device__ __forceinline__ int tile_cut(int j, int tiles, int n, int lg) {
    return tiles <= kEvenTiles ? j * n / tiles : min(j << lg, n);
}

// Totals -> scans, execution order, tile tables, host mail.  L.cnt[] and L.nbt[] hold the tokens and
// the batches of every expert on entry (behind a barrier).  Latency-bound (one workgroup): one
// thread per expert, prefix sums over the threads, and the tables written by 2^lt threads per
// expert.  (Thread 0 walking experts and tiles one by one made the scan of 64 experts take 27 us of a
// 52 us plan; the whole plan of 3072 assignments to 64 experts now takes 11 us in one launch.)
template <int T>
__device__ __forceinline__ void scan_body(const Shape& s, const PlanPtrs& p, int max_tiles, ScanLds& L) {
    static_assert(T >= kMaxExperts && T % 64 == 0, "one thread per expert");
    const int E = s.E, tid = threadIdx.x;
    const int c = tid < E ? L.cnt[tid] : 0;
    // order of execution: batches desc, tokens desc, index asc; 0 = not activated
    const unsigned long long key =
        c > 0 ? ((unsigned long long)L.nbt[tid] << 40) | ((unsigned long long)c << 8) | (unsigned)(255 - tid) : 0ull;
    if (tid < E) {
        L.key[tid] = key;
        L.ord[tid] = -1;
    }
    int o = c, po = (c + kRowBlk - 1) / kRowBlk * kRowBlk, total, ptotal;
    scan2(o, po, total, ptotal, L.wsum);
    if (tid < E) {
        L.off[tid] = o;
        L.pof[tid] = po;
    }
    if (tid == 0) {
        L.off[E] = total;
        L.pof[E] = ptotal;
    }
    __syncthreads();
    if (c > 0) {
        int rank = 0;
#pragma unroll 8
        for (int q = 0; q < E; ++q) rank += L.key[q] > key ? 1 : 0;
        L.ord[rank] = tid;
    }
    __syncthreads();
    // tiles: shared experts first (they serve every batch), then routed in execution order
    const int routed_blks = ptotal / kRowBlk, nblk_tok = (s.N + kRowBlk - 1) / kRowBlk;
    const int lg = s.tile_lg, last = (1 << lg) - 1;  // a tile is up to 2^lg row blocks
    const int per_shared = (nblk_tok + last) >> lg, shared_tiles = s.S * per_shared;
    const int mine = tid < E ? L.ord[tid] : -1;  // expert at place tid of the order
    const int nb = mine >= 0 ? (L.cnt[mine] + kRowBlk - 1) / kRowBlk : 0;
    int t0 = (nb + last) >> lg, place = mine >= 0 ? 1 : 0, routed_tiles, nact;
    scan2(t0, place, routed_tiles, nact, L.wsum);
    t0 += shared_tiles;
    const int nt = min(shared_tiles + routed_tiles, max_tiles);
    if (tid < E) {
        p.counts[tid] = c;
        p.offsets[tid] = o;
        p.poff[tid] = po;
        p.nbatch[tid] = L.nbt[tid];
        p.exec_order[tid] = mine;
        p.mail[tid] = c;
        p.mail[E + tid] = mine;
        if (p.out_counts) p.out_counts[tid] = c;
        if (p.out_offsets) p.out_offsets[tid] = o;
        if (p.out_exec_order) p.out_exec_order[tid] = mine;
        if (mine >= 0) {
            p.exp_tile0[mine] = t0;
            p.exp_ntiles[mine] = max(0, min((nb + last) >> lg, max_tiles - t0));
        }
        if (c == 0) {
            p.exp_tile0[tid] = 0;
            p.exp_ntiles[tid] = 0;
        }
    }
    if (tid < s.S) {
        p.exp_tile0[E + tid] = tid * per_shared;
        p.exp_ntiles[E + tid] = max(0, min(per_shared, max_tiles - tid * per_shared));
    }
    if (tid == 0) {
        p.offsets[E] = total;
        if (p.out_offsets) p.out_offsets[E] = total;
        p.poff[E] = ptotal;
        p.mail[2 * E] = nact;
        p.meta[0] = nact;
        p.meta[1] = nt;
        p.meta[2] = routed_blks;
        p.meta[3] = s.N;
    }
    // 2^lt threads write the row blocks of an expert and the tiles of a place of the order
    const int lt = 31 - __clz(T / E), part = tid & ((1 << lt) - 1), owner = tid >> lt;
    // the order's first tiles: handed over through LDS (key[] has been read by all)
    if (tid < E) L.key[tid] = (unsigned long long)t0;
    __syncthreads();
    if (owner < E) {
        const int b0 = L.pof[owner] / kRowBlk, blocks = (L.cnt[owner] + kRowBlk - 1) / kRowBlk;
        for (int b = part; b < blocks; b += 1 << lt) p.blk_expert[b0 + b] = owner;
        const int e = L.ord[owner];
        if (e >= 0) {
            const int x0 = L.pof[e] / kRowBlk, n = (L.cnt[e] + kRowBlk - 1) / kRowBlk, first = (int)L.key[owner];
            const int tiles = (n + last) >> lg;
            auto cut = [&](int j) { return tile_cut(j, tiles, n, lg); };
            for (int i = part; i < tiles && first + i < max_tiles; i += 1 << lt) {
                const int x = cut(i);
                p.tile_expert[first + i] = e;
                p.tile_xblk[first + i] = x0 + x;
                p.tile_hblk[first + i] = x0 + x;
                p.tile_nblk[first + i] = cut(i + 1) - x;
            }
        }
    }
    for (int i = tid; i < shared_tiles && i < max_tiles; i += T) {
        const int sh = i / per_shared, j = i - sh * per_shared, b = tile_cut(j, per_shared, nblk_tok, lg);
        p.tile_expert[i] = E + sh;
        p.tile_xblk[i] = routed_blks + b;
        p.tile_hblk[i] = routed_blks + sh * nblk_tok + b;
        p.tile_nblk[i] = tile_cut(j + 1, per_shared, nblk_tok, lg) - b;
    }
}

// P2: one block.  Sums the per-chunk histograms, then scan_body.  The chunk histograms pass through
// LDS in panels of kScanPanel entries (whole chunks): all threads load a panel (coalesced), one
// thread per expert runs down its column in LDS, all threads store the exclusive bases.  (One
// thread per expert walking global memory chunk by chunk took 34 us on a 32-chunk layer: a chain
// of dependent loads.)
constexpr int kScanPanel = 4096;
__global__ __launch_bounds__(kThreads) void plan_scan_kernel(Shape s, int nchunks, PlanPtrs p,
                                                             int max_tiles) {
    __shared__ ScanLds L;
    __shared__ int32_t panel[kScanPanel];
    __shared__ unsigned long long pmask[kMaxExperts];
    static_assert(kScanPanel >= kMaxExperts, "a panel holds at least one chunk");
    const int E = s.E;
    for (int e = threadIdx.x; e < E; e += kThreads) {
        L.cnt[e] = 0;
        pmask[e] = 0ull;
    }
    __syncthreads();
    const int per_panel = kScanPanel / E;  // whole chunks per panel
    for (int c0 = 0; c0 < nchunks; c0 += per_panel) {
        const int nc = min(per_panel, nchunks - c0);
        const size_t g0 = (size_t)c0 * E;
        for (int i = threadIdx.x; i < nc * E; i += kThreads) panel[i] = p.blk_counts[g0 + i];
        // batch masks: or-reduced per expert (order-free)
        for (int i = threadIdx.x; i < nc * E; i += kThreads) {
            const unsigned long long m = p.blk_mask[g0 + i];
            if (m) atomicOr(&pmask[i % E], m);
        }
        __syncthreads();
        for (int e = threadIdx.x; e < E; e += kThreads) {
            int run = L.cnt[e];
            for (int c = 0; c < nc; ++c) {
                const int v = panel[c * E + e];
                panel[c * E + e] = run;
                run += v;
            }
            L.cnt[e] = run;
        }
        __syncthreads();
        for (int i = threadIdx.x; i < nc * E; i += kThreads) p.blk_base[g0 + i] = panel[i];
        __syncthreads();
    }
    for (int e = threadIdx.x; e < E; e += kThreads) L.nbt[e] = __popcll(pmask[e]);
    __syncthreads();
    scan_body<kThreads>(s, p, max_tiles, L);
}

__device__ __forceinline__ void put_rank(const PlanPtrs& p, int a, int pos) {
    p.inv_perm[a] = pos;
    p.perm[pos] = a;
    if (p.out_inv_perm) p.out_inv_perm[a] = pos;
    if (p.out_perm) p.out_perm[pos] = a;
}

// P3: one block per chunk: stable position of every assignment of the chunk inside its expert's group.
__global__ __launch_bounds__(kThreads) void plan_rank_kernel(const int32_t* __restrict__ idx, int A,
                                                             int E, PlanPtrs p) {
    __shared__ int32_t seg[kSegs][kMaxExperts];  // tokens of expert e in (round, wave) segment
    __shared__ int32_t base[kMaxExperts];        // position of the chunk's first token of expert e
    const int wave = threadIdx.x >> 6, a0 = blockIdx.x * kPlanChunk;
    int my_e[kRounds], my_rank[kRounds];
#pragma unroll
    for (int r = 0; r < kRounds; ++r) {
        const int a = a0 + r * kThreads + threadIdx.x;
        my_e[r] = a < A ? idx[a] : -1;
    }
    for (int e = threadIdx.x; e < E; e += kThreads) {
        base[e] = p.offsets[e] + p.blk_base[(size_t)blockIdx.x * E + e];
#pragma unroll
        for (int sg = 0; sg < kSegs; ++sg) seg[sg][e] = 0;
    }
    __syncthreads();
    const int ebits = bits_for(E);
#pragma unroll
    for (int r = 0; r < kRounds; ++r) {
        const unsigned long long same = same_expert(my_e[r], ebits);
        my_rank[r] = __popcll(same & lanes_below());
        if (my_e[r] >= 0 && my_rank[r] == 0) seg[r * (kThreads / 64) + wave][my_e[r]] = __popcll(same);
    }
    __syncthreads();
    for (int e = threadIdx.x; e < E; e += kThreads) {  // exclusive scan over the 16 segments
        int run = base[e];
#pragma unroll
        for (int sg = 0; sg < kSegs; ++sg) {
            const int c = seg[sg][e];
            seg[sg][e] = run;
            run += c;
        }
    }
    __syncthreads();
#pragma unroll
    for (int r = 0; r < kRounds; ++r) {
        if (my_e[r] >= 0) {
            const int a = a0 + r * kThreads + threadIdx.x;
            const int pos = seg[r * (kThreads / 64) + wave][my_e[r]] + my_rank[r];
            put_rank(p, a, pos);
        }
    }
}

// All three phases in one block of T threads, for batch groups of up to kFusedRounds * T assignments.
// The counts are the sums of the wavefront segments that the ranks need anyway, so nothing but the
// batch masks goes through LDS atomics.  Up to 512 assignments take 256 threads: starting and joining
// twelve more wavefronts costs more than they save (gate and plan of 8 experts, 16 to 256 assignments 13.6
// us with 1024 threads, 12.3 with 256; 512 13.7 and 13.5; 1024 14.1 and 14.7).
constexpr int kFusedThreads = 1024, kFusedRounds = 4, kFusedMax = kFusedThreads * kFusedRounds;
template <int T>
__global__ __launch_bounds__(T) void plan_fused_kernel(const int32_t* __restrict__ idx, Shape s, BatchOffsets bo,
                                                       PlanPtrs p, int max_tiles, int rounds) {
    constexpr int kWaves = T / 64;
    __shared__ ScanLds L;
    __shared__ unsigned long long msk[kMaxExperts];
    __shared__ uint16_t seg[kFusedRounds * kWaves][kMaxExperts];  // tokens of expert e in (round, wave) segment
    __shared__ int32_t sbo[kMaxBatches + 1];
    const int A = s.N * s.k, E = s.E, wave = threadIdx.x >> 6, segs = rounds * kWaves;
    int my_e[kFusedRounds], my_rank[kFusedRounds];
#pragma unroll
    for (int r = 0; r < kFusedRounds; ++r) {
        const int a = r * T + threadIdx.x;
        my_e[r] = a < A ? idx[a] : -1;
    }
    if (threadIdx.x <= kMaxBatches) sbo[threadIdx.x] = bo.v[threadIdx.x];
    for (int i = threadIdx.x; i < segs * E; i += T) seg[i / E][i % E] = 0;
    if (threadIdx.x < E) msk[threadIdx.x] = 0ull;
    __syncthreads();
    const int ebits = bits_for(E);
#pragma unroll
    for (int r = 0; r < kFusedRounds; ++r) {
        my_rank[r] = 0;
        if (r < rounds) {  // uniform
            const int a = r * T + threadIdx.x, e = my_e[r];
            const unsigned long long same = same_expert(e, ebits);
            my_rank[r] = __popcll(same & lanes_below());
            if (e >= 0 && my_rank[r] == 0) seg[r * kWaves + wave][e] = (uint16_t)__popcll(same);
            add_batch(msk, e, a < A ? batch_of(sbo, bo.n, a / s.k) : 0, same);
        }
    }
    __syncthreads();
    if (threadIdx.x < E) {  // exclusive scan over the segments, its total the expert's tokens
        int run = 0;
#pragma unroll 8
        for (int sg = 0; sg < segs; ++sg) {
            const int c = seg[sg][threadIdx.x];
            seg[sg][threadIdx.x] = (uint16_t)run;
            run += c;
        }
        L.cnt[threadIdx.x] = run;
        L.nbt[threadIdx.x] = __popcll(msk[threadIdx.x]);
    }
    __syncthreads();
    scan_body<T>(s, p, max_tiles, L);
#pragma unroll
    for (int r = 0; r < kFusedRounds; ++r) {
        if (my_e[r] >= 0) {
            const int a = r * T + threadIdx.x;
            const int pos = L.off[my_e[r]] + seg[r * kWaves + wave][my_e[r]] + my_rank[r];
            put_rank(p, a, pos);
        }
    }
}

// Correlation table update (paper Section 6.2, path length 1): one thread per token adds its
// k x k (previous expert, current expert) pairs to the layer's table.  Integer atomics: the
// result does not depend on the order.
__global__ __launch_bounds__(kThreads) void corr_update_kernel(const int32_t* __restrict__ idx_prev,
                                                               const int32_t* __restrict__ idx_cur,
                                                               int N, int k, int E,
                                                               int32_t* __restrict__ table) {
    const int t = blockIdx.x * kThreads + threadIdx.x;
    if (t >= N) return;
    for (int a = 0; a < k; ++a) {
        const int p = idx_prev[(size_t)t * k + a];
        for (int b = 0; b < k; ++b) atomicAdd(&table[(size_t)p * E + idx_cur[(size_t)t * k + b]], 1);
    }
}

}  // namespace

void launch_corr_update(hipStream_t st, const int32_t* idx_prev, const int32_t* idx_cur, int N, int k,
                        int E, int32_t* table) {
    if (N <= 0) return;
    hipLaunchKernelGGL(corr_update_kernel, dim3((N + kThreads - 1) / kThreads), dim3(kThreads), 0, st,
                       idx_prev, idx_cur, N, k, E, table);
}

void launch_plan(hipStream_t st, const Shape& s, const BatchOffsets& bo, const PlanPtrs& p,
                 int max_tiles) {
    const int A = s.N * s.k;
    if (A <= 2 * kThreads) {
        hipLaunchKernelGGL(plan_fused_kernel<kThreads>, dim3(1), dim3(kThreads), 0, st, p.topk_idx, s, bo, p,
                           max_tiles, (A + kThreads - 1) / kThreads);
        return;
    }
    if (A <= kFusedMax) {
        hipLaunchKernelGGL(plan_fused_kernel<kFusedThreads>, dim3(1), dim3(kFusedThreads), 0, st, p.topk_idx, s, bo, p,
                           max_tiles, (A + kFusedThreads - 1) / kFusedThreads);
        return;
    }
    const int nchunks = (A + kPlanChunk - 1) / kPlanChunk;
    hipLaunchKernelGGL(plan_count_kernel, dim3(nchunks), dim3(kThreads), 0, st, p.topk_idx, A, s.E, s.k, bo,
                       p.blk_counts, p.blk_mask);
    hipLaunchKernelGGL(plan_scan_kernel, dim3(1), dim3(kThreads), 0, st, s, nchunks, p, max_tiles);
    hipLaunchKernelGGL(plan_rank_kernel, dim3(nchunks), dim3(kThreads), 0, st, p.topk_idx, A, s.E, p);
}

}  // namespace kmoe
