// Router: gate logits in a fixed fp32 summation order, wavefront top-k, routing weights.
//
// The gating network scores every expert for every token and the k best are activated
// (paper Section 2.1).  One 64-lane wavefront serves one token.  The logit of (token, expert)
// is accumulated in an order that a scalar program can reproduce exactly: the row is cut into
// 16-byte vectors, vector c belongs to lane c mod 64, a lane folds its elements in increasing
// index with fused multiply-adds, and the 64 partial sums meet in an xor butterfly
// (32,16,...,1).  IEEE addition is commutative, so every lane ends with the same value.
#include "kernels.h"

namespace kmoe {
namespace {

constexpr int kRouterWaves = 2;
constexpr int kCB = 4;  // vectors per lane loaded together
constexpr int kEG = 8;  // experts accumulated together

template <typename T>
struct Chunk;

template <>
struct Chunk<float> {
    static constexpr int V = 4;
    typedef float4 Raw;
    static __device__ __forceinline__ Raw raw(const float* p) { return *reinterpret_cast<const float4*>(p); }
    static __device__ __forceinline__ void widen(const Raw q, float (&v)[4]) {
        v[0] = q.x; v[1] = q.y; v[2] = q.z; v[3] = q.w;
    }
    static __device__ __forceinline__ void load(const float* p, float (&v)[4]) { widen(raw(p), v); }
};

struct bf16raw {
    uint16_t bits;
};

template <>
struct Chunk<bf16raw> {
    static constexpr int V = 8;
    typedef uint4 Raw;
    static __device__ __forceinline__ Raw raw(const bf16raw* p) { return *reinterpret_cast<const uint4*>(p); }
    static __device__ __forceinline__ void load(const bf16raw* p, float (&v)[8]) { widen(raw(p), v); }
    static __device__ __forceinline__ void widen(const Raw q, float (&v)[8]) {
        const uint32_t w[4] = {q.x, q.y, q.z, q.w};
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            v[2 * i] = __uint_as_float(w[i] << 16);            // low half = lower index
            v[2 * i + 1] = __uint_as_float(w[i] & 0xffff0000u);
        }
    }
};

struct Cand {
    float v;
    int e;  // -1: none
};

__device__ __forceinline__ bool better(const Cand& a, const Cand& b) {
    if (a.e < 0) return false;
    if (b.e < 0) return true;
    return a.v > b.v || (a.v == b.v && a.e < b.e);
}

__device__ __forceinline__ void put_winner(const RouterOut& out, size_t at, int e, float w) {
    out.idx[at] = e;
    out.w[at] = w;
    if (out.idx2) out.idx2[at] = e;
    if (out.w2) out.w2[at] = w;
}

// Top-k by (logit desc, index asc) and the routing weights of one token; every lane holds in
// mine[s] the logit of expert lane + 64 s.  One wavefront.
__device__ __forceinline__ void select_and_write(const float (&mine)[4], int lane, int t, int E, int k,
                                                 int renorm, const RouterOut& out) {
    bool taken[4] = {false, false, false, false};
    float selv[kMaxTopK];
    int sele[kMaxTopK];
#pragma unroll
    for (int j = 0; j < kMaxTopK; ++j) {
        selv[j] = 0.f;
        sele[j] = 0;
        if (j < k) {
            Cand best{0.f, -1};
#pragma unroll
            for (int s = 0; s < 4; ++s) {
                const int e = lane + 64 * s;
                Cand c{mine[s], (e < E && !taken[s]) ? e : -1};
                if (better(c, best)) best = c;
            }
#pragma unroll
            for (int m = 32; m >= 1; m >>= 1) {
                Cand o{__shfl_xor(best.v, m, 64), __shfl_xor(best.e, m, 64)};
                if (better(o, best)) best = o;
            }
            best.v = __shfl(best.v, 0, 64);
            best.e = __shfl(best.e, 0, 64);
            selv[j] = best.v;
            sele[j] = best.e;
#pragma unroll
            for (int s = 0; s < 4; ++s)
                if (best.e == lane + 64 * s) taken[s] = true;
        }
    }

    // routing weights: softmax over all experts, renormalised over the winners (or not)
    const float mx = selv[0];
    float den = 0.f;
    if (renorm) {
#pragma unroll
        for (int j = 0; j < kMaxTopK; ++j)
            if (j < k) den += expf(selv[j] - mx);
    } else {
#pragma unroll
        for (int s = 0; s < 4; ++s)
            if (lane + 64 * s < E) den += expf(mine[s] - mx);
#pragma unroll
        for (int m = 32; m >= 1; m >>= 1) den += __shfl_xor(den, m, 64);
    }
    if (lane == 0) {
#pragma unroll
        for (int j = 0; j < kMaxTopK; ++j) {
            if (j < k) {
                put_winner(out, (size_t)t * k + j, sele[j], expf(selv[j] - mx) / den);
            }
        }
    }
}

// The same for at most 64 experts with renormalised weights (v = the logit of expert `lane`): the rank
// of every expert is counted instead of selecting k times with a wavefront arg-max (12 dependent
// cross-lane moves through LDS per winner: at k = 6 half of the time of a 64-expert router).  Ranks
// come from a total order on (logit, index): the logit's bits mapped to an unsigned integer that
// grows with it, zeros of both signs alike.  No logit is NaN.
__device__ __forceinline__ void rank_and_write(float v, int lane, int t, int E, int k, const RouterOut& out) {
    const uint32_t u = __float_as_uint(v + 0.f);  // -0 -> +0
    // lanes without an expert: below every key, and behind every expert on a tie
    const uint32_t key = lane >= E ? 0u : u & 0x80000000u ? ~u : u | 0x80000000u;
    int rank = 0;
    for (int e0 = 0; e0 < E; e0 += 8) {
#pragma unroll
        for (int e = e0; e < e0 + 8; ++e) {
            const uint32_t o = __builtin_amdgcn_readlane(key, e);
            rank += o > key || (o == key && e < lane) ? 1 : 0;
        }
    }
    if (lane >= E) rank = 64;
    const unsigned long long first = __ballot(rank == 0);
    const float mx = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(v), __ffsll((long long)first) - 1));
    const float ex = expf(v - mx);
    float den = 0.f;
    for (int j = 0; j < k; ++j) {  // in order of rank
        const unsigned long long w = __ballot(rank == j);
        den += __int_as_float(__builtin_amdgcn_readlane(__float_as_int(ex), __ffsll((long long)w) - 1));
    }
    if (rank < k) put_winner(out, (size_t)t * k + rank, lane, ex / den);
}

// Sum over the 64 lanes of eight values at once, in the order of the xor butterfly (32, 16, ..., 1)
// stated at the top.  At step m a lane only needs lane[l] + lane[l ^ m] for the values it will
// still hold afterwards, so the lanes split the values between them: after the steps 32, 16 and
// 8 lane l holds value (l >> 3) & 7 alone, and the steps 4, 2, 1 finish it.  Each sum a lane
// forms is the one the full butterfly forms in that lane (IEEE addition is commutative), so the
// totals are bit for bit the butterfly's: 10 cross-lane moves instead of 48.  Returns the eight
// totals, uniform over the wavefront.
__device__ __forceinline__ void butterfly8(const float (&a)[kEG], int lane, float (&tot)[kEG]) {
    static_assert(kEG == 8, "three halving steps");
    float b[4], c[2], dsum;
    const bool h5 = (lane & 32) != 0, h4 = (lane & 16) != 0, h3 = (lane & 8) != 0;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        const float keep = h5 ? a[4 + i] : a[i], send = h5 ? a[i] : a[4 + i];
        b[i] = keep + __shfl_xor(send, 32, 64);
    }
#pragma unroll
    for (int i = 0; i < 2; ++i) {
        const float keep = h4 ? b[2 + i] : b[i], send = h4 ? b[i] : b[2 + i];
        c[i] = keep + __shfl_xor(send, 16, 64);
    }
    {
        const float keep = h3 ? c[1] : c[0], send = h3 ? c[0] : c[1];
        dsum = keep + __shfl_xor(send, 8, 64);
    }
#pragma unroll
    for (int m = 4; m >= 1; m >>= 1) dsum = dsum + __shfl_xor(dsum, m, 64);
#pragma unroll
    for (int j = 0; j < kEG; ++j)
        tot[j] = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(dsum), 8 * j));
}

// Top-k and renormalised routing weights of one token with at most kEG experts, from logits that
// are uniform over the wavefront: every lane selects for itself (no cross-lane traffic), lane 0
// writes.  Same order (logit descending, index ascending) and the same weight arithmetic as
// select_and_write with renorm set.
__device__ __forceinline__ void select_uniform_and_write(const float (&lg)[kEG], int E, int lane, int t,
                                                         int k, const RouterOut& out) {
    unsigned taken = 0u;
    float selv[kMaxTopK];
    int sele[kMaxTopK];
#pragma unroll
    for (int j = 0; j < kMaxTopK; ++j) {
        selv[j] = 0.f;
        sele[j] = 0;
        if (j < k) {
            int best = -1;
            float bv = 0.f;
#pragma unroll
            for (int e = 0; e < kEG; ++e) {
                const bool free_e = e < E && ((taken >> e) & 1u) == 0u;
                if (free_e && (best < 0 || lg[e] > bv)) {
                    best = e;
                    bv = lg[e];
                }
            }
            taken |= 1u << best;
            selv[j] = bv;
            sele[j] = best;
        }
    }
    const float mx = selv[0];
    float den = 0.f;
#pragma unroll
    for (int j = 0; j < kMaxTopK; ++j)
        if (j < k) den += expf(selv[j] - mx);
    if (lane == 0) {
#pragma unroll
        for (int j = 0; j < kMaxTopK; ++j) {
            if (j < k) {
                put_winner(out, (size_t)t * k + j, sele[j], expf(selv[j] - mx) / den);
            }
        }
    }
}

template <typename T>
__global__ __launch_bounds__(kRouterWaves * 64) void router_kernel(
    const T* __restrict__ X, const T* __restrict__ Wg, int N, int d, int E, int k, int renorm,
    RouterOut out) {
    constexpr int V = Chunk<T>::V;
    const int lane = threadIdx.x & 63;
    const int t = blockIdx.x * kRouterWaves + (threadIdx.x >> 6);
    if (t >= N) return;  // whole wavefront leaves; no block-wide synchronisation below
    const int nchunk = d / V;
    const T* xrow = X + (size_t)t * d;

    float mine[4];  // logits of experts lane, lane+64, lane+128, lane+192
#pragma unroll
    for (int s = 0; s < 4; ++s) mine[s] = 0.f;

    const int cpl = (nchunk + 63) / 64;  // vectors per lane
    for (int e0 = 0; e0 < E; e0 += kEG) {
        float acc[kEG];
#pragma unroll
        for (int j = 0; j < kEG; ++j) acc[j] = 0.f;
        // kCB vectors per lane at a time: all their loads are independent and issued together,
        // the fused multiply-adds then run in increasing element index per (expert, lane)
        for (int c0 = 0; c0 < cpl; c0 += kCB) {
            float xv[kCB][V];
#pragma unroll
            for (int q = 0; q < kCB; ++q) {
                const int c = (c0 + q) * 64 + lane;
                if (c < nchunk) {
                    Chunk<T>::load(xrow + (size_t)c * V, xv[q]);
                } else {
#pragma unroll
                    for (int i = 0; i < V; ++i) xv[q][i] = 0.f;
                }
            }
#pragma unroll
            for (int j = 0; j < kEG; ++j) {
                if (e0 + j < E) {
                    float wv[kCB][V];
#pragma unroll
                    for (int q = 0; q < kCB; ++q) {
                        const int c = min((c0 + q) * 64 + lane, nchunk - 1);  // clamped: x is 0 there
                        Chunk<T>::load(Wg + (size_t)(e0 + j) * d + (size_t)c * V, wv[q]);
                    }
#pragma unroll
                    for (int q = 0; q < kCB; ++q) {
                        if ((c0 + q) * 64 + lane < nchunk) {
#pragma unroll
                            for (int i = 0; i < V; ++i)
                                acc[j] = __builtin_fmaf(xv[q][i], wv[q][i], acc[j]);
                        }
                    }
                }
            }
        }
        float tot[kEG];
        butterfly8(acc, lane, tot);
#pragma unroll
        for (int j = 0; j < kEG; ++j) {
            const int e = e0 + j;
            if (e < E) {
                if (out.logits != nullptr && lane == 0) out.logits[(size_t)t * E + e] = tot[j];
                if ((e & 63) == lane) {
#pragma unroll
                    for (int s = 0; s < 4; ++s)
                        if ((e >> 6) == s) mine[s] = tot[j];
                }
            }
        }
        if (E <= kEG && renorm) {  // one group holds every expert: select in registers
            select_uniform_and_write(tot, E, lane, t, k, out);
            return;
        }
    }

    select_and_write(mine, lane, t, E, k, renorm, out);
}


// The same arithmetic for large batch groups of exactly kEG experts: one wavefront serves kMT tokens at a
// time, so that every vector of the gate matrix it loads (and widens) feeds kMT tokens, and the loop
// body has no branch: it serves shapes in which every lane holds a whole number of kMCB-vector groups
// (anything else takes router_kernel), so all loads of a group are in flight together.  Per (token,
// expert, lane) the order of the fused multiply-adds is the one stated at the top.  Tokens past the
// end re-read the last row and write nothing.
constexpr int kMT = 4;   // tokens per wavefront
constexpr int kMCB = 2;  // vectors per lane loaded together

// Adds to acc[q][j] the products of the MT token rows and kEG gate rows whose lane parts start at
// xrow[q] and wrow, cpl vectors per lane (a multiple of kMCB).
template <typename T, int MT>
__device__ __forceinline__ void score_group(const T* const (&xrow)[MT], const T* wrow, int d, int cpl,
                                            float (&acc)[MT][kEG]) {
    constexpr int V = Chunk<T>::V;
#pragma unroll
    for (int q = 0; q < MT; ++q)
#pragma unroll
        for (int j = 0; j < kEG; ++j) acc[q][j] = 0.f;
    for (int c0 = 0; c0 < cpl; c0 += kMCB) {
        typename Chunk<T>::Raw xr[MT][kMCB], wr[kEG][kMCB];
#pragma unroll
        for (int q = 0; q < MT; ++q)
#pragma unroll
            for (int b = 0; b < kMCB; ++b) xr[q][b] = Chunk<T>::raw(xrow[q] + (size_t)(c0 + b) * 64 * V);
#pragma unroll
        for (int j = 0; j < kEG; ++j)
#pragma unroll
            for (int b = 0; b < kMCB; ++b)
                wr[j][b] = Chunk<T>::raw(wrow + (size_t)j * d + (size_t)(c0 + b) * 64 * V);
#pragma unroll
        for (int b = 0; b < kMCB; ++b) {
            float xv[MT][V];
#pragma unroll
            for (int q = 0; q < MT; ++q) Chunk<T>::widen(xr[q][b], xv[q]);
#pragma unroll
            for (int j = 0; j < kEG; ++j) {
                float wv[V];
                Chunk<T>::widen(wr[j][b], wv);
#pragma unroll
                for (int q = 0; q < MT; ++q)
#pragma unroll
                    for (int i = 0; i < V; ++i) acc[q][j] = __builtin_fmaf(xv[q][i], wv[i], acc[q][j]);
            }
        }
    }
}

template <typename T>
__global__ __launch_bounds__(kRouterWaves * 64) void router_multi_kernel(
    const T* __restrict__ X, const T* __restrict__ Wg, int N, int d, int E, int k, int renorm,
    RouterOut out) {
    constexpr int V = Chunk<T>::V;
    const int lane = threadIdx.x & 63;
    const int t0 = (blockIdx.x * kRouterWaves + (threadIdx.x >> 6)) * kMT;
    if (t0 >= N) return;  // whole wavefront leaves; no block-wide synchronisation below
    const T* xrow[kMT];
#pragma unroll
    for (int q = 0; q < kMT; ++q) xrow[q] = X + (size_t)min(t0 + q, N - 1) * d + (size_t)lane * V;
    float acc[kMT][kEG];
    score_group<T, kMT>(xrow, Wg + (size_t)lane * V, d, d / (V * 64), acc);
#pragma unroll
    for (int q = 0; q < kMT; ++q) {
        float tot[kEG];
        butterfly8(acc[q], lane, tot);
        if (t0 + q >= N) continue;
        if (out.logits != nullptr && lane == 0)
#pragma unroll
            for (int j = 0; j < kEG; ++j) out.logits[(size_t)(t0 + q) * E + j] = tot[j];
        if (renorm) {
            select_uniform_and_write(tot, E, lane, t0 + q, k, out);
        } else {
            float mine[4] = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int j = 0; j < kEG; ++j)
                if (lane == j) mine[0] = tot[j];
            select_and_write(mine, lane, t0 + q, E, k, renorm, out);
        }
    }
}

// The same arithmetic for more than kEG experts: a workgroup of up to kWW wavefronts serves MT tokens and
// its wavefronts share the experts, kEG at a time, so that a gate vector is loaded once per MT tokens and
// no wavefront walks all experts (shapes as for router_multi_kernel).  The logits meet in LDS and the
// wavefronts select for the tokens.  Bound by the gate's re-reads from L2 and by latency: 512 tokens,
// 64 experts, width 2048 took 24-36 us with one token per workgroup (134 MB of gate rows).
constexpr int kWW = 8;
template <typename T, int MT>
__global__ __launch_bounds__(kWW * 64) void router_wide_kernel(
    const T* __restrict__ X, const T* __restrict__ Wg, int N, int d, int E, int k, int renorm,
    RouterOut out) {
    constexpr int V = Chunk<T>::V;
    __shared__ float slog[MT][kMaxExperts];
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
    const int waves = blockDim.x / 64;
    const int t0 = blockIdx.x * MT;
    const int cpl = d / (V * 64);  // vectors per lane, a multiple of kMCB
    const T* xrow[MT];
#pragma unroll
    for (int q = 0; q < MT; ++q) xrow[q] = X + (size_t)min(t0 + q, N - 1) * d + (size_t)lane * V;
    for (int e0 = wave * kEG; e0 < E; e0 += waves * kEG) {
        float acc[MT][kEG];
        score_group<T, MT>(xrow, Wg + (size_t)e0 * d + (size_t)lane * V, d, cpl, acc);
#pragma unroll
        for (int q = 0; q < MT; ++q) {
            float tot[kEG];
            butterfly8(acc[q], lane, tot);
#pragma unroll
            for (int j = 0; j < kEG; ++j)  // lane j of the group keeps the logit of expert e0 + j
                if (lane == j) {
                    slog[q][e0 + j] = tot[j];
                    if (out.logits != nullptr && t0 + q < N) out.logits[(size_t)(t0 + q) * E + e0 + j] = tot[j];
                }
        }
    }
    __syncthreads();
    auto select = [&](int q) {
        if (E <= 64 && renorm) {
            const float v = lane < E ? slog[q][lane] : 0.f;
            if (__ballot(v != v) == 0ull) {  // NaN has no place in the order of ranks: selected as everywhere else
                rank_and_write(v, lane, t0 + q, E, k, out);
                return;
            }
        }
        float mine[4];
#pragma unroll
        for (int s4 = 0; s4 < 4; ++s4) mine[s4] = lane + 64 * s4 < E ? slog[q][lane + 64 * s4] : 0.f;
        select_and_write(mine, lane, t0 + q, E, k, renorm, out);
    };
    if (MT <= 2) {  // there are at least two wavefronts
        if (wave < MT && t0 + wave < N) select(wave);
    } else {
        for (int q = wave; q < MT && t0 + q < N; q += waves) select(q);
    }
}

// The same arithmetic with one workgroup per token: wavefront w scores experts w*kSG, w*kSG+1,
// then (w+kSW)*kSG, ...; the token's row stays in registers (at most kSC vectors per lane) and
// the loads of a group's gate rows are all in flight together.  Logits meet in LDS and the first
// wavefront selects.  Used for small batch groups, where one wavefront per token leaves most
// of the chip idle.  The summation order per (token, expert) is the one stated at the top.
constexpr int kSW = 4;   // wavefronts per token
constexpr int kSG = 2;   // experts scored together by a wavefront
constexpr int kSC = 16;  // vectors of the row per lane, at most (template parameter SC: 2, 8 or 16)
template <typename T, int SC>
__global__ __launch_bounds__(kSW * 64) void router_split_kernel(
    const T* __restrict__ X, const T* __restrict__ Wg, int N, int d, int E, int k, int renorm,
    RouterOut out) {
    constexpr int V = Chunk<T>::V;
    __shared__ float slog[kMaxExperts];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int t = blockIdx.x;
    const int nchunk = d / V;
    const int cpl = (nchunk + 63) / 64;
    const T* xrow = X + (size_t)t * d;
    typename Chunk<T>::Raw xr[SC];  // the token's row, as stored; lanes past the end re-read the last vector
#pragma unroll
    for (int q = 0; q < SC; ++q)
        if (q < cpl) xr[q] = Chunk<T>::raw(xrow + (size_t)min(q * 64 + lane, nchunk - 1) * V);
    for (int e0 = wave * kSG; e0 < E; e0 += kSW * kSG) {
        // all gate vectors of the group are requested before the first multiply-add
        typename Chunk<T>::Raw wr[kSG][SC];
#pragma unroll
        for (int j = 0; j < kSG; ++j) {
            const int e = min(e0 + j, E - 1);  // clamped: the result of a surplus expert is dropped
#pragma unroll
            for (int q = 0; q < SC; ++q)
                if (q < cpl) wr[j][q] = Chunk<T>::raw(Wg + (size_t)e * d + (size_t)min(q * 64 + lane, nchunk - 1) * V);
        }
        float acc[kSG];
#pragma unroll
        for (int j = 0; j < kSG; ++j) {
            acc[j] = 0.f;
#pragma unroll
            for (int q = 0; q < SC; ++q) {
                if (q < cpl && q * 64 + lane < nchunk) {
                    float wv[V], xv[V];
                    Chunk<T>::widen(wr[j][q], wv);
                    Chunk<T>::widen(xr[q], xv);
#pragma unroll
                    for (int i = 0; i < V; ++i) acc[j] = __builtin_fmaf(xv[i], wv[i], acc[j]);
                }
            }
        }
#pragma unroll
        for (int j = 0; j < kSG; ++j) {
#pragma unroll
            for (int m = 32; m >= 1; m >>= 1) acc[j] = acc[j] + __shfl_xor(acc[j], m, 64);
            const int e = e0 + j;
            if (e < E && lane == 0) {
                slog[e] = acc[j];
                if (out.logits != nullptr) out.logits[(size_t)t * E + e] = acc[j];
            }
        }
    }
    __syncthreads();
    if (wave != 0) return;
    if (E <= kEG && renorm) {  // few experts: every lane reads them all and selects in registers
        float lg[kEG];
#pragma unroll
        for (int e = 0; e < kEG; ++e) lg[e] = e < E ? slog[e] : 0.f;
        select_uniform_and_write(lg, E, lane, t, k, out);
        return;
    }
    float mine[4];
#pragma unroll
    for (int s4 = 0; s4 < 4; ++s4) mine[s4] = lane + 64 * s4 < E ? slog[lane + 64 * s4] : 0.f;
    select_and_write(mine, lane, t, E, k, renorm, out);
}

}  // namespace

void launch_router(hipStream_t st, int dtype, const void* x, const void* wg, const Shape& s,
                   const RouterOut& out) {
    if (s.N <= 0) return;
    const int V = dtype == 0 ? 4 : 8;
    const int cpl = (s.d / V + 63) / 64;
    // more experts than one group: the tokens of a workgroup share the gate rows.  Few tokens spread over
    // more workgroups instead (one token each below 256, two below 1024)
    if (dtype != 0 && s.d % (8 * 64 * kMCB) == 0 && s.E % kEG == 0 && s.E > kEG) {
        const int mt = s.N < 256 ? 1 : s.N < 1024 ? 2 : 4;
        // Wavefronts per workgroup: no more than there are groups of experts (idle ones would only hold
        // registers: 16 experts, width 4096, 8192 tokens 79 us with eight, 35 with two), but below 2048
        // tokens one per token to select (1500 tokens 17.1 us with two, 15.9 with four, 23.3 with eight).
        // From 2048 tokens on the workgroups no longer run all at once, and up to four wavefronts that walk
        // the groups in even passes use the chip better (64 experts, width 2048, eight against four: 1024
        // tokens 15 and 20 us, 2048 24 and 23, 8192 73 and 61).
        const int groups = s.E / kEG, most = s.N < 2048 ? kWW : kWW / 2, passes = (groups + most - 1) / most;
        const int few = groups < mt ? mt : groups < most ? groups : most;
        const int waves = s.N < 2048 ? few : (groups + passes - 1) / passes;
        const dim3 grid((s.N + mt - 1) / mt), block(waves * 64);
#define KMOE_WIDE(MT)                                                                                     \
    hipLaunchKernelGGL((router_wide_kernel<bf16raw, MT>), grid, block, 0, st, (const bf16raw*)x,            \
                       (const bf16raw*)wg, s.N, s.d, s.E, s.k, s.renorm, out)
        if (mt == 1) KMOE_WIDE(1); else if (mt == 2) KMOE_WIDE(2); else KMOE_WIDE(4);
#undef KMOE_WIDE
        return;
    }
    if (s.N <= 2048 && cpl <= kSC) {  // small batch group: one workgroup per token
        dim3 grid(s.N), block(kSW * 64);
#define KMOE_SPLIT(T, SC)                                                                              \
    hipLaunchKernelGGL((router_split_kernel<T, SC>), grid, block, 0, st, (const T*)x, (const T*)wg, s.N, \
                       s.d, s.E, s.k, s.renorm, out)
        if (dtype == 0) {
            if (cpl <= 2) KMOE_SPLIT(float, 2); else if (cpl <= 8) KMOE_SPLIT(float, 8); else KMOE_SPLIT(float, 16);
        } else {
            if (cpl <= 2) KMOE_SPLIT(bf16raw, 2); else if (cpl <= 8) KMOE_SPLIT(bf16raw, 8); else KMOE_SPLIT(bf16raw, 16);
        }
#undef KMOE_SPLIT
        return;
    }
    // large bf16 batch groups of a shape the branch-free kernel serves: kMT tokens share every gate vector
    if (dtype != 0 && s.N >= 8192 && s.d % (8 * 64 * kMCB) == 0 && s.E == kEG) {
        const int per_block = kRouterWaves * kMT;
        dim3 grid((s.N + per_block - 1) / per_block), block(kRouterWaves * 64);
        hipLaunchKernelGGL(router_multi_kernel<bf16raw>, grid, block, 0, st, (const bf16raw*)x,
                           (const bf16raw*)wg, s.N, s.d, s.E, s.k, s.renorm, out);
        return;
    }
    dim3 grid((s.N + kRouterWaves - 1) / kRouterWaves), block(kRouterWaves * 64);
    if (dtype == 0) {
        hipLaunchKernelGGL(router_kernel<float>, grid, block, 0, st, (const float*)x,
                           (const float*)wg, s.N, s.d, s.E, s.k, s.renorm, out);
    } else {
        hipLaunchKernelGGL(router_kernel<bf16raw>, grid, block, 0, st, (const bf16raw*)x,
                           (const bf16raw*)wg, s.N, s.d, s.E, s.k, s.renorm, out);
    }
}

}  // namespace kmoe
