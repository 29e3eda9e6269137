// fp32 expert FFN (SwiGLU) for the fp32 configuration, on the fp32 matrix instruction.
//
// Each expert is an FFN applied to the tokens routed to it (paper Section 2.1); rows follow
// the same padded per-expert row space and the same tiles as the bf16 path.  A workgroup takes up
// to 64 rows of one expert (two row blocks of a tile) and UN units of 32 weight rows; a unit of the
// up projection stacks 16 rows of W1 on the same 16 of W3, so that the gate and the up value of a
// feature meet in one lane.  The four wavefronts are NB row blocks x UN units x KS parts of the
// reduction.  fp32 operands and products (32x32x2 MFMA, one fused multiply-add per product), accurate
// expf; chains of eight products, pairs of chains added in fp32, the rest of the sum in fp64.  That
// rounds a dot product of any length less than 64 lanes that stride it and meet in a tree do: relative
// error of the layer against 64 bits, in 1e-7, 64 x 64 1.32 (64 lanes: 1.42), 256 x 512 1.34 (1.58),
// 1024 x 256 1.33 (1.78), 1024 x 2048 1.40 (2.06), 2048 x 4096 1.48 (2.56).  (Chains of 16 and fp32 sums
// above them: 1.59, 1.78, 1.91, 2.04, 2.31, and 4 % faster; fp32 sums above chains of 8: as fast as
// those, 1.41, 1.70, 1.82, 1.96, 2.23.)
//
// What bounds it: the matrix instruction, and with few rows per expert the expert weights.  A
// workgroup per row with a dot product per wavefront read every weight once per row: the layer of
// 256 tokens, top-2 of 8 experts, 1024 x 2048 took 844 (up) + 774 us (down); in tiles it takes 71 + 53 us
// (60 and 41 TFLOP/s, padding rows not counted).  Both operands pass through LDS (straight from the
// row-major matrices, 32 bytes of 32 rows per load, they took twice as long): whole 128-byte lines from
// memory, double buffered, the 16-byte pieces of a row permuted by the row's number so that the reads
// of 16 rows spread over the 64 banks.
#include <type_traits>

#include "kernels.h"

namespace kmoe {
namespace {

typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
// Rows are read through pointers marked as global memory: activations and weights come from
// different bases, and loads of an unknown address space (flat) would count as LDS traffic too, so
// that every wait for LDS also waited for the stages in flight.
typedef const __attribute__((address_space(1))) f32x4* gvec;

constexpr int kWaves = 4, kThr = kWaves * 64;
constexpr int kSliceK = 32;           // reduction elements of one wavefront and stage: a 128-byte line per row
constexpr int kPieces = kSliceK / 4;  // 16-byte pieces of a row's slice
constexpr int kPairBlks = 2;          // row blocks per workgroup, at most
constexpr int kPairsPerTile = kTileBlks / kPairBlks;

template <int NB, int UN>
struct Geo {
    static constexpr int KS = kWaves / (NB * UN);         // parts of the reduction
    static constexpr int ROWS = (NB + UN) * 32;           // operand rows of a stage: activations, then weights
    static constexpr int LOADS = ROWS * kPieces * KS / kThr;  // 16-byte loads per thread and stage
    static constexpr int STAGE = ROWS * kPieces * KS;     // 16-byte pieces of a stage
};

// Sums over the whole reduction (K elements, a multiple of 4) of one workgroup.  row(r) is operand
// row r (activations 0 .. NB*32-1, then weights).  Valid on return for wavefronts with ks == 0:
// register i holds, of the wavefront's unit and row block, weight row 8 (i / 4) + 4 (lane / 32) + i % 4
// and activation row lane % 32 (WFIRST) or the other way round.
template <int NB, int UN, bool WFIRST, typename RowFn>
__device__ __forceinline__ f32x16 reduce_tile(RowFn row, int K, f32x4* lds) {
    using G = Geo<NB, UN>;
    static_assert(NB * UN * G::KS == kWaves && G::ROWS * kPieces * G::KS % kThr == 0, "geometry");
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
    const int b = wave % NB, u = wave / NB % UN, ks = wave / (NB * UN);
    // a thread's loads: piece threadIdx % 8 of rows threadIdx / 8 + 32 i, slice by slice
    const int piece = threadIdx.x % kPieces, r0 = threadIdx.x / kPieces;
    constexpr int RL = NB + UN;  // loads of a slice
    gvec src[RL];
#pragma unroll
    for (int i = 0; i < RL; ++i) src[i] = (gvec)(uintptr_t)(row(r0 + 32 * i)) + piece;
    typedef f32x4 Regs[G::LOADS];
    constexpr int kStageK = kSliceK * G::KS;
    // Loads never branch (the waits below count them); pieces past the end read the row's start and
    // are replaced by zeros when they go to LDS.  whole: the stage has no such piece.
    auto load = [&](Regs& x, int k0, auto whole) {
#pragma unroll
        for (int sl = 0; sl < G::KS; ++sl) {
            const int k = k0 + sl * kSliceK;
            const int at = decltype(whole)::value || k + piece * 4 < K ? k / 4 : -piece;  // -piece: the row's start
#pragma unroll
            for (int i = 0; i < RL; ++i) x[sl * RL + i] = src[i][at];
        }
    };
    auto slot = [](int sl, int r, int pc) { return (sl * G::ROWS + r) * kPieces + (pc ^ ((r >> 1) & (kPieces - 1))); };
    auto store = [&](const Regs& x, int k0, int buf, auto whole) {
#pragma unroll
        for (int sl = 0; sl < G::KS; ++sl) {
            const bool in = decltype(whole)::value || k0 + sl * kSliceK + piece * 4 < K;
#pragma unroll
            for (int i = 0; i < RL; ++i)
                lds[buf * G::STAGE + slot(sl, r0 + 32 * i, piece)] = in ? x[sl * RL + i] : f32x4{0.f, 0.f, 0.f, 0.f};
        }
    };
    double total[16];
#pragma unroll
    for (int i = 0; i < 16; ++i) total[i] = 0.;
    // Stage k0 from LDS buffer `buf`; the next one goes from x to the other buffer, and x is filled with
    // the third.  Two stages are in flight because one stage's 1024 cycles of MFMA are shorter than
    // the memory latency.  steady: all of that exists and is whole, so there is no branch and the
    // wait before the stores leaves the younger loads in flight.
    auto stage = [&](Regs& x, int k0, int buf, auto steady) {
        if (decltype(steady)::value || k0 + kStageK < K) store(x, k0 + kStageK, buf ^ 1, steady);
        if (decltype(steady)::value || k0 + 3 * kStageK < K) load(x, k0 + 3 * kStageK, steady);
        const f32x4* L = lds + buf * G::STAGE;
        f32x4 xa[kPieces / 2], wa[kPieces / 2];
#pragma unroll
        for (int st = 0; st < kPieces / 2; ++st) {  // the lane's half of a step of eight elements
            const int pc = 2 * st + (lane >> 5);
            xa[st] = L[slot(ks, b * 32 + (lane & 31), pc)];
            wa[st] = L[slot(ks, (NB + u) * 32 + (lane & 31), pc)];
        }
        f32x16 acc[2];  // two chains of eight products per half stage
#pragma unroll
        for (int half = 0; half < 2; ++half) {
#pragma unroll
            for (int st = 2 * half; st < 2 * half + 2; ++st)
#pragma unroll
                for (int j = 0; j < 4; ++j)
                    acc[j & 1] = __builtin_amdgcn_mfma_f32_32x32x2f32(WFIRST ? wa[st][j] : xa[st][j], WFIRST ? xa[st][j] : wa[st][j],
                                                                      st % 2 == 0 && j < 2 ? f32x16{} : acc[j & 1], 0, 0, 0);
#pragma unroll
            for (int i = 0; i < 16; ++i) total[i] += (double)(acc[0][i] + acc[1][i]);
        }
        __syncthreads();
    };
    Regs xa, xb;
    load(xa, 0, std::false_type{});
    store(xa, 0, 0, std::false_type{});
    load(xa, kStageK, std::false_type{});
    load(xb, 2 * kStageK, std::false_type{});
    __syncthreads();
    int k0 = 0;
    for (; k0 + 5 * kStageK <= K; k0 += 2 * kStageK) {
        stage(xa, k0, 0, std::true_type{});
        stage(xb, k0 + kStageK, 1, std::true_type{});
    }
    for (; k0 < K; k0 += 2 * kStageK) {
        stage(xa, k0, 0, std::false_type{});
        if (k0 + kStageK < K) stage(xb, k0 + kStageK, 1, std::false_type{});  // uniform over the workgroup
    }
    if (G::KS > 1) {  // the parts of the reduction are added in order (LDS: behind the last barrier)
        double* red = reinterpret_cast<double*>(lds);
        const int tile = wave % (NB * UN);
        if (ks > 0)
#pragma unroll
            for (int i = 0; i < 16; ++i) red[(((ks - 1) * NB * UN + tile) * 16 + i) * 64 + lane] = total[i];
        __syncthreads();
        if (ks == 0)
#pragma unroll
            for (int p = 0; p < G::KS - 1; ++p)
#pragma unroll
                for (int i = 0; i < 16; ++i) total[i] += red[((p * NB * UN + tile) * 16 + i) * 64 + lane];
    }
    f32x16 sums;
#pragma unroll
    for (int i = 0; i < 16; ++i) sums[i] = (float)total[i];
    return sums;
}

// Grid: (groups of output features, row parts, the parts beyond kGridY in z).  Features come first, so
// that the workgroups of a row part spread over all XCDs and those that share weight rows (the parts of
// an expert) tend to meet on one: parts first took 1.8 times as long.
constexpr int kGridY = 32768;

struct Part {
    int e, hblk, nblk;  // expert, first row block of H and O, live row blocks (1 or 2; 0: nothing here)
    int xblk;           // first row block in the token space of the expert
};

// Which expert and row blocks does this workgroup serve?  Only the parts that exist are numbered, tile by
// tile (sums over the tile table, a tile per lane).  A tile has up to four parts, mostly one or two, and
// workgroups go to the compute units in turn whatever these hold already: with all four numbered some units
// held three live workgroups and others none, by the multiples of the feature groups.  Layers, four
// numbered / those that exist, top-2: 8 experts of 1024 x 2048, 8 tokens 92 / 72 us, 128 139 / 92, 256 141 /
// 140, 512 222 / 228, 4096 1118 / 1123; 12 of 256 x 1536, 264 tokens 84 / 69; 128 + 2 of 512 x 256, top-6, 512 tokens 225 / 133.
// (Two wavefronts per SIMD, the additions between the MFMAs of the next half stage, evened the placement out
// by accident and helped or hurt by the same multiples; with the parts in a row three wavefronts are
// as fast or faster at every size.)
__device__ __forceinline__ Part locate(const PlanPtrs& p, int only_expert, int max_tiles) {
    static_assert(kPairsPerTile < 8, "three bits per tile");
    Part w{0, 0, 0, 0};
    const int lane = threadIdx.x & 63;
    const int tile0 = only_expert >= 0 ? p.exp_tile0[only_expert] : 0;
    const int tiles = min(only_expert >= 0 ? p.exp_ntiles[only_expert] : p.meta[1], max_tiles);
    int part = (int)blockIdx.z * kGridY + (int)blockIdx.y;
    for (int t0 = 0; t0 < tiles; t0 += 64) {
        const int tile = tile0 + min(t0 + lane, max_tiles - 1);  // all loads at once, `tiles` included
        const int e = p.tile_expert[tile], hblk = p.tile_hblk[tile], xblk = p.tile_xblk[tile], nblk = p.tile_nblk[tile];
        const int n = t0 + lane < tiles ? (nblk + kPairBlks - 1) / kPairBlks : 0;
        const uint64_t ones = __ballot(n & 1), twos = __ballot(n & 2), fours = __ballot(n & 4);
        auto sum = [&](uint64_t lanes) {
            return __popcll(ones & lanes) + 2 * __popcll(twos & lanes) + 4 * __popcll(fours & lanes);
        };
        const int total = sum(~0ull);
        if (part < total) {
            const int pair = part - sum((1ull << lane) - 1);  // of this lane's tile, if it has as many
            const int l = __ffsll((unsigned long long)__ballot(pair >= 0 && pair < n)) - 1;
            auto of = [&](int v) { return __builtin_amdgcn_readlane(v, l); };
            const int first = of(pair) * kPairBlks;
            w.e = of(e);
            w.hblk = of(hblk) + first;
            w.xblk = of(xblk) + first;
            w.nblk = min(kPairBlks, of(nblk) - first);
            break;
        }
        part -= total;
    }
    return w;
}

// Token of row r of the workgroup's rows, -1 for padding.
__device__ __forceinline__ int token_of(const Shape& s, const PlanPtrs& p, const Part& w, int r) {
    if (w.e < s.E) {
        const int rank = w.xblk * kRowBlk + r - p.poff[w.e];
        return rank < p.counts[w.e] ? p.perm[p.offsets[w.e] + rank] / s.k : -1;
    }
    const int t = (w.xblk - p.meta[2]) * kRowBlk + r;  // shared experts: the tokens in order
    return t < s.N ? t : -1;
}

// h[row, n] = silu(W1[n,:] . x) * (W3[n,:] . x)
constexpr int kUpUnits = 2, kUpFeat = 16 * kUpUnits;
template <int NB>
__device__ __forceinline__ void up_rows(const float* __restrict__ x, const Shape& s, const PlanPtrs& p,
                                        const Part& w, const float* blob, f32x4* lds, float* __restrict__ h) {
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
    const int n0 = (int)blockIdx.x * kUpFeat;
    auto row = [&](int r) -> const float* {  // padding rows read token 0, features past the end the last one
        if (r < NB * 32) return x + (size_t)max(0, token_of(s, p, w, r)) * s.d;
        const int i = (r - NB * 32) % 32, n = min(n0 + (r - NB * 32) / 32 * 16 + i % 16, s.f - 1);
        return blob + ((size_t)(i / 16) * s.f + n) * s.d;
    };
    const f32x16 acc = reduce_tile<NB, kUpUnits, true>(row, s.d, lds);
    if (wave / (NB * kUpUnits) != 0) return;
    const int r = wave % NB * 32 + (lane & 31), f0 = n0 + wave / NB % kUpUnits * 16 + 4 * (lane >> 5);
    if (token_of(s, p, w, r) < 0) return;
    float* dst = h + ((size_t)w.hblk * kRowBlk + r) * s.f;
#pragma unroll
    for (int q = 0; q < 2; ++q) {  // registers 4q .. 4q+3: features f0 + 8q .. +3; the up values 8 registers on
        float v[4];
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const float g = acc[4 * q + j];
            v[j] = g / (1.f + expf(-g)) * acc[4 * q + j + 8];
        }
        if (f0 + 8 * q < s.f)  // f is a multiple of 4
            *reinterpret_cast<float4*>(dst + f0 + 8 * q) = make_float4(v[0], v[1], v[2], v[3]);
    }
}

// Wavefronts per SIMD (launch bounds): what LDS leaves room for; a few dwords per lane go to scratch.
// (Without the down projection's bound its accumulators went to AGPRs: layer above 148 us instead of 143.)
__global__ __launch_bounds__(kThr, 3) void ffn_up_f32_kernel(
    const float* __restrict__ x, Shape s, PlanPtrs p, const uint8_t* const* __restrict__ wtab,
    const uint8_t* __restrict__ w_single, int only_expert, int max_tiles, float* __restrict__ h) {
    __shared__ f32x4 lds[2 * Geo<1, kUpUnits>::STAGE];
    static_assert(Geo<1, kUpUnits>::STAGE >= Geo<2, kUpUnits>::STAGE, "LDS of the larger stage");
    const Part w = locate(p, only_expert, max_tiles);
    if (w.nblk == 0) return;
    const float* blob = reinterpret_cast<const float*>(w_single ? w_single : wtab[w.e]);
    if (w.nblk == 1)
        up_rows<1>(x, s, p, w, blob, lds, h);
    else
        up_rows<2>(x, s, p, w, blob, lds, h);
}

// o[row, m] = W2[m,:] . h[row,:]
constexpr int kDownUnits = 1, kDownFeat = 32 * kDownUnits;
template <int NB>
__device__ __forceinline__ void down_rows(const Shape& s, const Part& w, const float* w2, f32x4* lds,
                                          const float* __restrict__ h, float* __restrict__ o) {
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
    const int m0 = (int)blockIdx.x * kDownFeat;
    auto row = [&](int r) -> const float* {  // padding rows hold whatever is there: a row only reaches its own sums
        if (r < NB * 32) return h + ((size_t)w.hblk * kRowBlk + r) * s.f;
        return w2 + (size_t)min(m0 + r - NB * 32, s.d - 1) * s.f;
    };
    const f32x16 acc = reduce_tile<NB, kDownUnits, false>(row, s.f, lds);
    if (wave / (NB * kDownUnits) != 0) return;
    const int col = m0 + wave / NB % kDownUnits * 32 + (lane & 31);
    if (col >= s.d) return;
#pragma unroll
    for (int i = 0; i < 16; ++i) {
        const size_t r = (size_t)w.hblk * kRowBlk + wave % NB * 32 + 8 * (i / 4) + 4 * (lane >> 5) + i % 4;
        o[r * s.d + col] = acc[i];
    }
}

__global__ __launch_bounds__(kThr, 2) void ffn_down_f32_kernel(
    Shape s, PlanPtrs p, const uint8_t* const* __restrict__ wtab,
    const uint8_t* __restrict__ w_single, int only_expert, int max_tiles, const float* __restrict__ h,
    float* __restrict__ o) {
    __shared__ f32x4 lds[2 * Geo<1, kDownUnits>::STAGE];
    static_assert(Geo<1, kDownUnits>::STAGE >= Geo<2, kDownUnits>::STAGE, "LDS of the larger stage");
    const Part w = locate(p, only_expert, max_tiles);
    if (w.nblk == 0) return;
    const float* w2 = reinterpret_cast<const float*>(w_single ? w_single : wtab[w.e]) + 2 * (size_t)s.f * s.d;
    if (w.nblk == 1)
        down_rows<1>(s, w, w2, lds, h, o);
    else
        down_rows<2>(s, w, w2, lds, h, o);
}

}  // namespace

void launch_ffn_f32(hipStream_t st, const float* x, const Shape& s, const PlanPtrs& p,
                    const uint8_t* const* wtab, const uint8_t* w_single, int32_t only_expert,
                    int32_t max_tiles, float* h, float* o) {
    if (s.N <= 0 || max_tiles <= 0) return;
    auto grid = [&](int features, int per_group) {
        const int parts = max_tiles * kPairsPerTile;
        return dim3((features + per_group - 1) / per_group, parts < kGridY ? parts : kGridY, (parts + kGridY - 1) / kGridY);
    };
    hipLaunchKernelGGL(ffn_up_f32_kernel, grid(s.f, kUpFeat), dim3(kThr), 0, st, x, s, p, wtab, w_single,
                       only_expert, max_tiles, h);
    hipLaunchKernelGGL(ffn_down_f32_kernel, grid(s.d, kDownFeat), dim3(kThr), 0, st, s, p, wtab, w_single,
                       only_expert, max_tiles, h, o);
}

}  // namespace kmoe
