// Kernels of the attention (non-expert) layer for one decoding step of one batch.
//
// Algorithm 1 of the paper runs the non-expert layer batch by batch; the arithmetic is the
// attention layer of the paper's model family (Section 2.1) with its normalisation folded in
// (Section 4): RMS norm, q/k/v projections, rotary embedding, cache append, grouped-query
// softmax attention of the one new token over the cached positions, output projection and
// residual.  The projections are dense contractions and run on bf16 MFMA (32x32x16, fp32
// accumulate) with weights pre-packed in fragment order so that a wavefront streams one
// contiguous run of 1 KiB fragments; with few rows they are bound by the weight bytes, so the
// reduction is split across wavefronts until the chip is full and the partial sums are added in
// a fixed order by the kernel that consumes them.  The attention core is bound by the cache
// bytes: one workgroup per (sequence, key-value head) reads every K and V row once, 16 bytes
// per lane, all query heads of the group sharing each row.  Cache rows are read with
// non-temporal loads and the weights with ordinary ones: the layer's weights (tens of MB) are
// read again for every batch of the group and fit the last-level cache, the caches of a batch are
// read once and would only evict them.
#include <type_traits>

#include "attn_kernels.h"
#include "attn_ranges.h"

namespace kattn {
namespace {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));

__device__ __forceinline__ float bf_lo(uint32_t w) { return __uint_as_float(w << 16); }
__device__ __forceinline__ float bf_hi(uint32_t w) { return __uint_as_float(w & 0xffff0000u); }
__device__ __forceinline__ uint32_t bf_bits(float a) {
    return (uint32_t)__builtin_bit_cast(uint16_t, (__bf16)a);  // round to nearest even
}
__device__ __forceinline__ uint32_t pack2(float lo, float hi) { return bf_bits(lo) | (bf_bits(hi) << 16); }
__device__ __forceinline__ void widen8(const u32x4 v, float (&f)[8]) {
    f[0] = bf_lo(v.x); f[1] = bf_hi(v.x); f[2] = bf_lo(v.y); f[3] = bf_hi(v.y);
    f[4] = bf_lo(v.z); f[5] = bf_hi(v.z); f[6] = bf_lo(v.w); f[7] = bf_hi(v.w);
}
__device__ __forceinline__ bf16x8 as_bf16x8(const u32x4 v) { return __builtin_bit_cast(bf16x8, v); }

// 16-byte piece index of element (row, k) of a [rows, K] matrix in fragment order.
__device__ __forceinline__ size_t frag_piece(int row, int chunk, int S) {
    return ((size_t)(row >> 5) * S + (chunk >> 1)) * 64 + (row & 31) + 32 * (chunk & 1);
}

// Batch that owns activation row `row` (the table has at most kMaxGroup entries).
__device__ __forceinline__ int find_batch(const GroupTab& tab, int row) {
    int b = 0;
    while (b + 1 < tab.n && row >= tab.row0[b + 1]) ++b;
    return b;
}

__global__ __launch_bounds__(256) void pack_weight_kernel(const u32x4* __restrict__ w, int rows, int K,
                                                          u32x4* __restrict__ out) {
    const size_t i = (size_t)blockIdx.x * 256 + threadIdx.x;
    if (i >= (size_t)rows * K / 8) return;
    const int lane = (int)(i & 63), S = K / 16;
    const size_t unit = i >> 6;
    const int s = (int)(unit % S), rb = (int)(unit / S);
    const int row = rb * 32 + (lane & 31), k0 = s * 16 + (lane >> 5) * 8;
    out[i] = w[((size_t)row * K + k0) / 8];
}

// One workgroup per row; a thread keeps its 16-byte pieces of the row in registers between the
// sum of squares and the scaling (rows of up to 256 * 8 * kNormPieces elements).
constexpr int kNormPieces = 4;
__global__ __launch_bounds__(256) void rmsnorm_kernel(GroupTab tab, const u32x4* __restrict__ g, int d,
                                                      float eps, u32x4* __restrict__ a) {
    __shared__ float part[4];
    const int row = blockIdx.x, nch = d / 8, S = d / 16;
    const int bt = find_batch(tab, row);
    const u32x4* xr = (const u32x4*)tab.h_in[bt] + (size_t)(row - tab.row0[bt]) * nch;
    u32x4 xv[kNormPieces], gv[kNormPieces];
#pragma unroll
    for (int i = 0; i < kNormPieces; ++i) {
        const int c = threadIdx.x + i * 256;
        if (c < nch) {
            xv[i] = xr[c];
            gv[i] = g[c];
        }
    }
    float ss = 0.f;
#pragma unroll
    for (int i = 0; i < kNormPieces; ++i) {
        if (threadIdx.x + i * 256 < nch) {
            float f[8];
            widen8(xv[i], f);
#pragma unroll
            for (int j = 0; j < 8; ++j) ss = __builtin_fmaf(f[j], f[j], ss);
        }
    }
#pragma unroll
    for (int m = 32; m >= 1; m >>= 1) ss += __shfl_xor(ss, m, 64);
    if ((threadIdx.x & 63) == 0) part[threadIdx.x >> 6] = ss;
    __syncthreads();
    ss = (part[0] + part[1]) + (part[2] + part[3]);
    const float r = 1.0f / sqrtf(ss / (float)d + eps);
#pragma unroll
    for (int i = 0; i < kNormPieces; ++i) {
        const int c = threadIdx.x + i * 256;
        if (c < nch) {
            float f[8], gg[8];
            widen8(xv[i], f);
            widen8(gv[i], gg);
            u32x4 o;
            o.x = pack2(f[0] * r * gg[0], f[1] * r * gg[1]);
            o.y = pack2(f[2] * r * gg[2], f[3] * r * gg[3]);
            o.z = pack2(f[4] * r * gg[4], f[5] * r * gg[5]);
            o.w = pack2(f[6] * r * gg[6], f[7] * r * gg[7]);
            a[frag_piece(row, c, S)] = o;
        }
    }
}

// One wavefront per (U column blocks of 32 outputs, split of the reduction, row tile of NB
// blocks): every activation fragment it loads feeds U MFMAs, every weight fragment NB.
template <int NB, int U>
__global__ __launch_bounds__(256, 2) void proj_kernel(const u32x4* __restrict__ A,
                                                   const u32x4* __restrict__ W, float* __restrict__ out,
                                                   int S, int CB, int splits, int n_rt, int n_out,
                                                   int64_t split_stride) {
    const int lane = threadIdx.x & 63;
    const int w = blockIdx.x * 4 + (threadIdx.x >> 6);
    const int CG = CB / U;  // column groups (host-checked: U divides CB)
    if (w >= CG * splits * n_rt) return;
    const int cg = w % CG, sp = (w / CG) % splits, rt = w / (CG * splits);
    const int SS = S / splits;  // a multiple of 8 (host-checked)
    const u32x4* wp = W + ((size_t)cg * U * S + (size_t)sp * SS) * 64 + lane;
    const u32x4* ap = A + ((size_t)rt * NB * S + (size_t)sp * SS) * 64 + lane;
    constexpr int C = U == 1 ? 4 : 2;
    f32x16 acc[U][NB];
#pragma unroll
    for (int u = 0; u < U; ++u)
#pragma unroll
        for (int b = 0; b < NB; ++b)
#pragma unroll
            for (int r = 0; r < 16; ++r) acc[u][b][r] = 0.f;
    u32x4 w0[C][U], w1[C][U], a0[C][NB], a1[C][NB];
    auto load = [&](u32x4(&wb)[C][U], u32x4(&ab)[C][NB], int s) {
#pragma unroll
        for (int j = 0; j < C; ++j) {
#pragma unroll
            for (int u = 0; u < U; ++u) wb[j][u] = wp[((size_t)u * S + s + j) * 64];
#pragma unroll
            for (int b = 0; b < NB; ++b) ab[j][b] = ap[((size_t)b * S + s + j) * 64];
        }
    };
    auto mac = [&](const u32x4(&wb)[C][U], const u32x4(&ab)[C][NB]) {
#pragma unroll
        for (int j = 0; j < C; ++j)
#pragma unroll
            for (int b = 0; b < NB; ++b)
#pragma unroll
                for (int u = 0; u < U; ++u)
                    acc[u][b] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(as_bf16x8(ab[j][b]), as_bf16x8(wb[j][u]),
                                                                        acc[u][b], 0, 0, 0);
    };
    load(w0, a0, 0);
    for (int s = 0; s < SS; s += 2 * C) {
        load(w1, a1, s + C);
        mac(w0, a0);
        if (s + 2 * C < SS) load(w0, a0, s + 2 * C);
        mac(w1, a1);
    }
    float* o = out + (size_t)sp * split_stride;
#pragma unroll
    for (int u = 0; u < U; ++u) {
        const int col = (cg * U + u) * 32 + (lane & 31);
#pragma unroll
        for (int b = 0; b < NB; ++b)
#pragma unroll
            for (int r = 0; r < 16; ++r) {
                const size_t row = (size_t)(rt * NB + b) * kRowBlk + 8 * (r / 4) + 4 * (lane >> 5) + r % 4;
                o[row * n_out + col] = acc[u][b][r];
            }
    }
}

// One thread per rotated pair of FH consecutive heads of q and k (they share the angle, whose reduction,
// sine and cosine cost more than the sums), or per element of v, of one sequence.
template <int FH>
__global__ __launch_bounds__(256) void qkv_finish_kernel(const float* __restrict__ part, int splits,
                                                         int64_t split_stride, Dims dm, GroupTab tab,
                                                         const double* __restrict__ inv_freq,
                                                         float* __restrict__ q) {
    const int row_g = blockIdx.y, hd = dm.hd, half = hd / 2;
    const int bt = find_batch(tab, row_g);
    const int s = row_g - tab.row0[bt], n_seq = tab.row0[bt + 1] - tab.row0[bt], pos = tab.pos[bt];
    uint16_t* kc = (uint16_t*)tab.kc[bt];
    uint16_t* vc = (uint16_t*)tab.vc[bt];
    uint16_t* new_rows = (uint16_t*)tab.new_rows[bt];
    const int dq = dm.Hq * hd, dkv = dm.Hkv * hd, n_out = dq + 2 * dkv;
    const int heads = dm.Hq + dm.Hkv;  // heads 0..Hq-1 are q, then k
    const int n_pairs = (heads + FH - 1) / FH * half;
    const int i = blockIdx.x * 256 + threadIdx.x;
    if (i >= n_pairs + dkv) return;
    const float* row = part + (size_t)row_g * n_out;
    if (i < n_pairs) {
        const int h0 = i / half * FH, j = i % half;
        float a[FH], b[FH];
#pragma unroll
        for (int u = 0; u < FH; ++u) a[u] = b[u] = 0.f;
        for (int sp = 0; sp < splits; ++sp) {  // partial sums in order, all heads of a split side by side
            const float* p = row + (size_t)sp * split_stride + j;
#pragma unroll
            for (int u = 0; u < FH; ++u) {
                const int h = min(h0 + u, heads - 1);  // past the last head: the last one again, unused
                a[u] += p[h * hd];
                b[u] += p[h * hd + half];
            }
        }
        // angle reduced to [-pi, pi] in double, sine and cosine of the remainder in single
        const double ang = (double)pos * inv_freq[j];
        const double turns = rint(ang * 0.15915494309189535);
        const float red = (float)(ang - turns * 6.283185307179586);
        float sf, c;
        sincosf(red, &sf, &c);
#pragma unroll
        for (int u = 0; u < FH; ++u) {
            const int h = h0 + u;
            if (h >= heads) break;
            const float r0 = a[u] * c - b[u] * sf, r1 = b[u] * c + a[u] * sf;
            if (h < dm.Hq) {
                // 1/sqrt(hd) and log2(e) folded in: the attention kernel works with base-2 exponentials
                const float qscale = 1.4426950408889634f / sqrtf((float)hd);
                q[((size_t)row_g * dm.Hq + h) * hd + j] = r0 * qscale;
                q[((size_t)row_g * dm.Hq + h) * hd + j + half] = r1 * qscale;
            } else {
                const int hk = h - dm.Hq;
                const uint16_t b0 = (uint16_t)bf_bits(r0), b1 = (uint16_t)bf_bits(r1);
                uint16_t* dst = kc + (((size_t)s * dm.Hkv + hk) * dm.max_len + pos) * hd;
                dst[j] = b0;
                dst[j + half] = b1;
                if (new_rows != nullptr) {
                    uint16_t* nr = new_rows + ((size_t)s * dm.Hkv + hk) * hd;
                    nr[j] = b0;
                    nr[j + half] = b1;
                }
            }
        }
    } else {
        const int e = i - n_pairs, hk = e / hd, j = e % hd;
        float v = 0.f;
        for (int sp = 0; sp < splits; ++sp) v += row[(size_t)sp * split_stride + dq + dkv + e];
        const uint16_t b = (uint16_t)bf_bits(v);
        vc[(((size_t)s * dm.Hkv + hk) * dm.max_len + pos) * hd + j] = b;
        if (new_rows != nullptr) new_rows[((size_t)(n_seq + s) * dm.Hkv + hk) * hd + j] = b;
    }
}

// Sum over the LPR (4, 8 or 16) consecutive lanes that share a row, by data-parallel-primitive
// adds: lane pairs, quad halves, then the mirrored half row and the mirrored row (after the
// first two steps every quad holds one value, so a mirror acts as the xor exchange).
template <int LPR>
__device__ __forceinline__ float row_sum(float v) {
    auto dpp = [](float x, auto ctrl) {
        return __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, x), decltype(ctrl)::value, 0xF, 0xF, false));
    };
    v += dpp(v, std::integral_constant<int, 0xB1>{});                  // quad_perm [1,0,3,2]
    v += dpp(v, std::integral_constant<int, 0x4E>{});                  // quad_perm [2,3,0,1]
    if (LPR > 4) v += dpp(v, std::integral_constant<int, 0x141>{});    // row_half_mirror
    if (LPR > 8) v += dpp(v, std::integral_constant<int, 0x140>{});    // row_mirror
    return v;
}

struct Soft {  // running softmax (base 2) of one (query head, 8-element slice)
    float m, l, acc[8];
};
__device__ __forceinline__ void merge(Soft& a, float m2, float l2, const float (&acc2)[8]) {
    const float mn = fmaxf(a.m, m2);
    const float sa = __builtin_amdgcn_exp2f(a.m - mn), sb = __builtin_amdgcn_exp2f(m2 - mn);
    a.l = a.l * sa + l2 * sb;
#pragma unroll
    for (int j = 0; j < 8; ++j) a.acc[j] = a.acc[j] * sa + acc2[j] * sb;
    a.m = mn;
}

constexpr float kEmpty = -1.0e30f;  // finite stand-in for "no position seen yet"
// The reference of a running softmax follows the largest score only once a score exceeds it by this much
// (base 2): the sums are not rescaled chunk by chunk, and the weights stay below 2^kLag instead of 1.  Sums of
// values that reach kWide so (or are not finite) are formed again without the lag, by weights up to 1; below
// it the sums of all slots, wavefronts and ranges together stay finite.
constexpr float kLag = 8.f, kWide = 0x1p100f;

// Normalised output of 8 elements (16-byte chunk `chunk` of the row) as bf16 in fragment order.
template <int HD>
__device__ __forceinline__ void write_head(u32x4* __restrict__ o_frag, int row, int chunk, int Hq, const Soft& t) {
    const float inv = 1.0f / t.l;  // position pos is always valid, so l > 0
    u32x4 o;
    o.x = pack2(t.acc[0] * inv, t.acc[1] * inv);
    o.y = pack2(t.acc[2] * inv, t.acc[3] * inv);
    o.z = pack2(t.acc[4] * inv, t.acc[5] * inv);
    o.w = pack2(t.acc[6] * inv, t.acc[7] * inv);
    o_frag[frag_piece(row, chunk, Hq * HD / 16)] = o;
}

// One workgroup (4 wavefronts) per (sequence, key-value head, part of the cached positions); G query
// heads share the rows.  A row of HD elements is read by HD/8 lanes (16 bytes each); a wavefront
// covers 512/HD rows per load, issues the K and V loads of kChunk such row groups together, and keeps
// one running softmax per row slot (rescaled when its reference moves, see kLag), merged at the end.
//
// Bound by the cache bytes as long as the chip has loads in flight.  A few sequences with long
// caches do not fill it with one workgroup per (sequence, head): 4 sequences x 8 heads x 8000
// positions (6 query heads each) ran 32 workgroups for 920 us (0.14 TB/s; 284 bytes of scratch per
// lane came on top), so the positions of a batch's sequences are cut into equal ranges (attn_ranges):
// 23 ranges took 36 us (3.6 TB/s) and 5 us for the merge.  With six query heads the vector instructions of a
// row, not its bytes, are the limit: without the rescaling and the masks of chunk after chunk (a quarter of
// them) the layer takes 109 us instead of 115, 512 sequences of 500 positions 346 instead of 368.  A
// sequence of one range is written by its workgroup; with several each writes its unnormalised sums and
// attn_merge_kernel adds them up.  512 sequences x 8 heads x 513 positions keep one range: 173 us, 6.3 TB/s.
template <int HD, int G>
__global__ __launch_bounds__(kAttnWaves * 64, attn_waves_per_simd(G)) void attn_decode_kernel(
    const float* __restrict__ q, Dims dm, GroupTab tab, int all, RangeTab rt, float* __restrict__ part_acc,
    float2* __restrict__ part_ml, u32x4* __restrict__ o_frag) {
    constexpr int LPR = HD / 8, RPW = 64 / LPR;
    constexpr bool AHEAD = G > 4;
    __shared__ float sm[kAttnWaves][G * LPR][10];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    int bt = 0, ranges = all, in_batch = (int)blockIdx.x, row0 = 0;
    if (all == 0) {
        while (bt + 1 < tab.n && (int)blockIdx.x >= rt.first[bt + 1] * dm.Hkv) ++bt;
        ranges = rt.n[bt];
        in_batch -= rt.first[bt] * dm.Hkv;
        row0 = tab.row0[bt];
    }
    const int sp = in_batch % ranges, pair = in_batch / ranges;
    const int hk = pair % dm.Hkv, row_g = row0 + pair / dm.Hkv;
    if (all != 0) bt = find_batch(tab, row_g);
    const int s = row_g - tab.row0[bt];
    const int len = tab.pos[bt] + 1;  // positions 0..pos
    const int per = (len + ranges - 1) / ranges;
    const int first = sp * per, end = min(first + per, len);  // the last range may be empty
    const int sub = lane % LPR, slot = lane / LPR;
    float qr[G][8];
#pragma unroll
    for (int g = 0; g < G; ++g)
#pragma unroll
        for (int j = 0; j < 8; ++j) qr[g][j] = q[((size_t)row_g * dm.Hq + hk * G + g) * HD + sub * 8 + j];
    const size_t base = ((size_t)s * dm.Hkv + hk) * dm.max_len * LPR + sub;
    const u32x4* K = (const u32x4*)tab.kc[bt] + base;
    const u32x4* V = (const u32x4*)tab.vc[bt] + base;
    Soft st[G];
    // rows past the end re-read the range's last row (in bounds and at hand) and count as zeros
    auto load = [&](u32x4(&kr)[kChunk], u32x4(&vr)[kChunk], int p0) {
#pragma unroll
        for (int c = 0; c < kChunk; ++c) {
            const int p = min(p0 + c * RPW + slot, end - 1);
            kr[c] = __builtin_nontemporal_load(K + (size_t)p * LPR);
            vr[c] = __builtin_nontemporal_load(V + (size_t)p * LPR);
        }
    };
    constexpr int STEP = kAttnWaves * RPW * kChunk;
    int p0;
    u32x4 kraw[kChunk], vraw[kChunk], knext[kChunk], vnext[kChunk];
    // whole: every row of the chunk is in the range, so nothing is masked
    auto step = [&](auto whole, float lag) {
        if (AHEAD) {
#pragma unroll
            for (int c = 0; c < kChunk; ++c) {
                kraw[c] = knext[c];
                vraw[c] = vnext[c];
            }
            load(knext, vnext, p0 + STEP);
        } else {
            load(kraw, vraw, p0);
        }
        bool valid[kChunk];
#pragma unroll
        for (int c = 0; c < kChunk; ++c) valid[c] = decltype(whole)::value || p0 + c * RPW + slot < end;
        if (!decltype(whole)::value)  // weight 0 alone would make NaN of an infinite value
#pragma unroll
            for (int c = 0; c < kChunk; ++c)
                if (!valid[c]) vraw[c] = u32x4{0u, 0u, 0u, 0u};
        float sc[G][kChunk];
#pragma unroll
        for (int c = 0; c < kChunk; ++c) {
            float kf[8];
            widen8(kraw[c], kf);
#pragma unroll
            for (int g = 0; g < G; ++g) {
                float dot = 0.f;
#pragma unroll
                for (int j = 0; j < 8; ++j) dot = __builtin_fmaf(qr[g][j], kf[j], dot);
                dot = row_sum<LPR>(dot);
                sc[g][c] = valid[c] ? dot : kEmpty;
            }
        }
        float over = 0.f;  // how far the chunk's scores exceed the reference
#pragma unroll
        for (int g = 0; g < G; ++g) {
            float mn = sc[g][0];
#pragma unroll
            for (int c = 1; c < kChunk; ++c) mn = fmaxf(mn, sc[g][c]);
            over = fmaxf(over, mn - st[g].m);
        }
        if (__any(over > lag)) {
#pragma unroll
            for (int g = 0; g < G; ++g) {
                float mn = st[g].m;
#pragma unroll
                for (int c = 0; c < kChunk; ++c) mn = fmaxf(mn, sc[g][c]);
                const float sa = __builtin_amdgcn_exp2f(st[g].m - mn);
                st[g].l *= sa;
                st[g].m = mn;
#pragma unroll
                for (int j = 0; j < 8; ++j) st[g].acc[j] *= sa;
            }
        }
        float pr[G][kChunk];
#pragma unroll
        for (int g = 0; g < G; ++g)
#pragma unroll
            for (int c = 0; c < kChunk; ++c) {
                pr[g][c] = valid[c] ? __builtin_amdgcn_exp2f(sc[g][c] - st[g].m) : 0.f;
                st[g].l += pr[g][c];
            }
#pragma unroll
        for (int c = 0; c < kChunk; ++c) {
            float vf[8];
            widen8(vraw[c], vf);
#pragma unroll
            for (int g = 0; g < G; ++g)
#pragma unroll
                for (int j = 0; j < 8; ++j) st[g].acc[j] = __builtin_fmaf(pr[g][c], vf[j], st[g].acc[j]);
        }
    };
    auto begin = [&] {
#pragma unroll
        for (int g = 0; g < G; ++g) {
            st[g].m = kEmpty;
            st[g].l = 0.f;
#pragma unroll
            for (int j = 0; j < 8; ++j) st[g].acc[j] = 0.f;
        }
        p0 = first + wave * RPW * kChunk;
    };
    begin();
    if (AHEAD && p0 < end) load(knext, vnext, p0);
    for (; p0 + kChunk * RPW <= end; p0 += STEP) step(std::true_type{}, kLag);
    if (p0 < end) step(std::false_type{}, kLag);  // the wavefront's last rows
    float size = 0.f;  // a sum, so that NaN stays
#pragma unroll
    for (int g = 0; g < G; ++g)
#pragma unroll
        for (int j = 0; j < 8; ++j) size += fabsf(st[g].acc[j]);
    if (!__all(size < kWide)) {
        begin();
        for (; p0 < end; p0 += STEP) {
            if (AHEAD) load(knext, vnext, p0);
            step(std::false_type{}, 0.f);
        }
    }
    // row slots of the wavefront
#pragma unroll
    for (int off = LPR; off < 64; off <<= 1) {
#pragma unroll
        for (int g = 0; g < G; ++g) {
            const float m2 = __shfl_xor(st[g].m, off, 64), l2 = __shfl_xor(st[g].l, off, 64);
            float a2[8];
#pragma unroll
            for (int j = 0; j < 8; ++j) a2[j] = __shfl_xor(st[g].acc[j], off, 64);
            merge(st[g], m2, l2, a2);
        }
    }
    if (slot == 0) {
#pragma unroll
        for (int g = 0; g < G; ++g) {
            float* e = sm[wave][g * LPR + sub];
            e[0] = st[g].m;
            e[1] = st[g].l;
#pragma unroll
            for (int j = 0; j < 8; ++j) e[2 + j] = st[g].acc[j];
        }
    }
    __syncthreads();
    if (threadIdx.x < G * LPR) {
        const int g = threadIdx.x / LPR, sb = threadIdx.x % LPR;
        Soft t;
        t.m = kEmpty;
        t.l = 0.f;
#pragma unroll
        for (int j = 0; j < 8; ++j) t.acc[j] = 0.f;
#pragma unroll
        for (int w = 0; w < kAttnWaves; ++w) {
            const float* e = sm[w][threadIdx.x];
            float a2[8];
#pragma unroll
            for (int j = 0; j < 8; ++j) a2[j] = e[2 + j];
            merge(t, e[0], e[1], a2);
        }
        if (ranges > 1) {
            const size_t at = (size_t)((all != 0 ? row_g * all : rt.first[bt] + s * ranges) + sp) * dm.Hq + hk * G + g;
            float4* pa = reinterpret_cast<float4*>(part_acc + at * HD + sb * 8);
            pa[0] = make_float4(t.acc[0], t.acc[1], t.acc[2], t.acc[3]);
            pa[1] = make_float4(t.acc[4], t.acc[5], t.acc[6], t.acc[7]);
            if (sb == 0) part_ml[at] = make_float2(t.m, t.l);
            return;
        }
        write_head<HD>(o_frag, row_g, (hk * G + g) * LPR + sb, dm.Hq, t);
    }
}

// Adds up the ranges of one (row, query head): one wavefront, HD/8 lanes per range, so that 512/HD
// ranges are summed side by side (kMergeAhead of them requested before the first is used) and then
// merged over the lanes.  Latency-bound: with one thread per 8 elements walking all ranges 23 ranges
// took 10.4 us.
constexpr int kMergeAhead = 4;
template <int HD>
__global__ __launch_bounds__(256) void attn_merge_kernel(const float* __restrict__ part_acc,
                                                         const float2* __restrict__ part_ml, int rows, int Hq,
                                                         int all, u32x4* __restrict__ o_frag, GroupTab tab, RangeTab rt) {
    constexpr int LPR = HD / 8, SIDE = 64 / LPR;
    const int lane = threadIdx.x & 63, sub = lane % LPR;
    const int rh = blockIdx.x * 4 + (threadIdx.x >> 6), row = rh / Hq, head = rh % Hq;
    if (row >= rows) return;  // uniform over the wavefront
    int ranges = all;
    size_t first = (size_t)row * all;
    if (all == 0) {
        const int bt = find_batch(tab, row);
        ranges = rt.n[bt];
        first = (size_t)rt.first[bt] + (size_t)(row - tab.row0[bt]) * ranges;
        if (ranges == 1) return;
    }
    Soft t;
    t.m = kEmpty;
    t.l = 0.f;
#pragma unroll
    for (int j = 0; j < 8; ++j) t.acc[j] = 0.f;
    for (int s0 = lane / LPR; s0 < ranges; s0 += SIDE * kMergeAhead) {
        float2 ml[kMergeAhead];
        float4 lo[kMergeAhead], hi[kMergeAhead];
#pragma unroll
        for (int u = 0; u < kMergeAhead; ++u) {  // past the end: the last range again, unused
            const size_t at = (first + min(s0 + u * SIDE, ranges - 1)) * Hq + head;
            const float4* pa = reinterpret_cast<const float4*>(part_acc + at * HD + sub * 8);
            ml[u] = part_ml[at];
            lo[u] = pa[0];
            hi[u] = pa[1];
        }
#pragma unroll
        for (int u = 0; u < kMergeAhead; ++u) {
            if (s0 + u * SIDE >= ranges) break;
            const float a2[8] = {lo[u].x, lo[u].y, lo[u].z, lo[u].w, hi[u].x, hi[u].y, hi[u].z, hi[u].w};
            merge(t, ml[u].x, ml[u].y, a2);
        }
    }
#pragma unroll
    for (int off = LPR; off < 64; off <<= 1) {
        const float m2 = __shfl_xor(t.m, off, 64), l2 = __shfl_xor(t.l, off, 64);
        float a2[8];
#pragma unroll
        for (int j = 0; j < 8; ++j) a2[j] = __shfl_xor(t.acc[j], off, 64);
        merge(t, m2, l2, a2);
    }
    if (lane < LPR) write_head<HD>(o_frag, row, head * LPR + sub, Hq, t);
}

__global__ __launch_bounds__(256) void out_finish_kernel(const float* __restrict__ part, int splits,
                                                         int64_t split_stride, GroupTab tab, int d) {
    const size_t i = (size_t)blockIdx.x * 256 + threadIdx.x;  // 8 consecutive elements
    const int nch = d / 8;
    if (i >= (size_t)tab.row0[tab.n] * nch) return;
    const int row = (int)(i / nch), bt = find_batch(tab, row);
    const size_t at = (size_t)(row - tab.row0[bt]) * nch + i % nch;
    float f[8];
    widen8(((const u32x4*)tab.h_in[bt])[at], f);
    for (int sp = 0; sp < splits; ++sp) {
        const float4* p = reinterpret_cast<const float4*>(part + (size_t)sp * split_stride + i * 8);
        const float4 a = p[0], b = p[1];
        f[0] += a.x; f[1] += a.y; f[2] += a.z; f[3] += a.w;
        f[4] += b.x; f[5] += b.y; f[6] += b.z; f[7] += b.w;
    }
    u32x4 o;
    o.x = pack2(f[0], f[1]);
    o.y = pack2(f[2], f[3]);
    o.z = pack2(f[4], f[5]);
    o.w = pack2(f[6], f[7]);
    ((u32x4*)tab.h_out[bt])[at] = o;
}

}  // namespace

void launch_pack_weight(hipStream_t st, const void* w, int rows, int K, void* out) {
    const size_t pieces = (size_t)rows * K / 8;
    hipLaunchKernelGGL(pack_weight_kernel, dim3((unsigned)((pieces + 255) / 256)), dim3(256), 0, st,
                       (const u32x4*)w, rows, K, (u32x4*)out);
}

void launch_rmsnorm(hipStream_t st, const GroupTab& tab, const void* g, int d, float eps, void* a_frag) {
    hipLaunchKernelGGL(rmsnorm_kernel, dim3(tab.row0[tab.n]), dim3(256), 0, st, tab, (const u32x4*)g, d, eps,
                       (u32x4*)a_frag);
}

int pick_row_tile(int row_blocks) { return row_blocks >= 3 ? 4 : row_blocks == 2 ? 2 : 1; }

// Column blocks per wavefront: two once a row tile is full (128 rows), where the activation
// fragments re-read from L2 are what the kernel moves most of.
static int pick_col_units(int row_blocks, int n_out) { return row_blocks >= 4 && (n_out / 32) % 2 == 0 ? 2 : 1; }

int pick_splits(int row_blocks, int K, int n_out) {
    const int U = pick_col_units(row_blocks, n_out);
    const int S = K / 16, CG = n_out / 32 / U;
    const int nb = pick_row_tile(row_blocks), n_rt = (row_blocks + nb - 1) / nb;
    int splits = 1;
    while (splits < kMaxSplit && CG * n_rt * splits < (U == 2 ? 768 : 1024) && S % (splits * 2 * 8) == 0) splits *= 2;
    return splits;
}

void launch_proj(hipStream_t st, const void* a_frag, const void* w_frag, int row_blocks, int K,
                 int n_out, int splits, float* out, int64_t split_stride) {
    const int S = K / 16, CB = n_out / 32;
    const int nb = pick_row_tile(row_blocks), n_rt = (row_blocks + nb - 1) / nb;
    const int U = pick_col_units(row_blocks, n_out);
    const int waves = CB / U * splits * n_rt;
    const dim3 grid((waves + 3) / 4), block(256);
    const u32x4* A = (const u32x4*)a_frag;
    const u32x4* W = (const u32x4*)w_frag;
    if (nb == 4 && U == 2)
        hipLaunchKernelGGL((proj_kernel<4, 2>), grid, block, 0, st, A, W, out, S, CB, splits, n_rt, n_out, split_stride);
    else if (nb == 4)
        hipLaunchKernelGGL((proj_kernel<4, 1>), grid, block, 0, st, A, W, out, S, CB, splits, n_rt, n_out, split_stride);
    else if (nb == 2)
        hipLaunchKernelGGL((proj_kernel<2, 1>), grid, block, 0, st, A, W, out, S, CB, splits, n_rt, n_out, split_stride);
    else
        hipLaunchKernelGGL((proj_kernel<1, 1>), grid, block, 0, st, A, W, out, S, CB, splits, n_rt, n_out, split_stride);
}

// Heads per thread: one, which is done soonest, while the chip holds all workgroups at once (eight of 256
// threads per compute unit); then two, which share the angle.  (32/8 heads of 128: 16 rows 3.3 us with one
// head, 3.5 with two, 4.0 with four; 512 rows 9.1, 7.7 and 7.2; 48/8 heads 128 rows 8.7, 6.2 and 10.4; 32/8
// heads of 32, 64 rows 3.4, 3.6 and 5.1.)
void launch_qkv_finish(hipStream_t st, const float* part, int splits, int64_t split_stride,
                       const Dims& dm, const GroupTab& tab, const double* inv_freq, float* q) {
    const int rows = tab.row0[tab.n], heads = dm.Hq + dm.Hkv;
    auto blocks = [&](int FH) { return ((heads + FH - 1) / FH * (dm.hd / 2) + dm.Hkv * dm.hd + 255) / 256; };
    const int FH = rows * blocks(1) <= 256 * 8 ? 1 : 2;
    const dim3 grid(blocks(FH), rows), block(256);
    if (FH == 1)
        hipLaunchKernelGGL(qkv_finish_kernel<1>, grid, block, 0, st, part, splits, split_stride, dm, tab, inv_freq, q);
    else
        hipLaunchKernelGGL(qkv_finish_kernel<2>, grid, block, 0, st, part, splits, split_stride, dm, tab, inv_freq, q);
}

template <int HD>
static int launch_attention_hd(hipStream_t st, const float* q, const Dims& dm, const GroupTab& tab,
                               float* scratch, int max_ranges, void* o_frag) {
    const int rows = tab.row0[tab.n], G = dm.Hq / dm.Hkv;
    RangeTab rt;
    rt.first[0] = 0;
    bool cut = false, same = true;
    for (int b = 0; b < tab.n; ++b) {
        rt.n[b] = b > 0 && tab.pos[b] == tab.pos[b - 1] ? rt.n[b - 1]
                                                        : attn_ranges(tab.pos[b] + 1, (long)rows * dm.Hkv, G, HD, max_ranges);
        rt.first[b + 1] = rt.first[b] + (tab.row0[b + 1] - tab.row0[b]) * rt.n[b];
        cut = cut || rt.n[b] > 1;
        same = same && rt.n[b] == rt.n[0];
    }
    // the number of ranges if it is the same everywhere: the kernels then need not look it up first (each
    // look-up is a wait on the arguments, about 0.5 us in kernels of 5)
    const int all = same ? rt.n[0] : 0;
    const int items = rt.first[tab.n];
    const dim3 grid(items * dm.Hkv), block(kAttnWaves * 64);
    u32x4* O = (u32x4*)o_frag;
    float2* ml = (float2*)(scratch + (size_t)items * dm.Hq * HD);
    switch (G) {
#define KATTN_CASE(G) \
    case G: hipLaunchKernelGGL((attn_decode_kernel<HD, G>), grid, block, 0, st, q, dm, tab, all, rt, scratch, ml, O); break;
        KATTN_CASE(1) KATTN_CASE(2) KATTN_CASE(3) KATTN_CASE(4) KATTN_CASE(5) KATTN_CASE(6) KATTN_CASE(7) KATTN_CASE(8)
#undef KATTN_CASE
        default: return -1;
    }
    if (cut)
        hipLaunchKernelGGL(attn_merge_kernel<HD>, dim3((rows * dm.Hq + 3) / 4), dim3(256), 0, st,
                           scratch, ml, rows, dm.Hq, all, O, tab, rt);
    return 0;
}

int launch_attention(hipStream_t st, const float* q, const Dims& dm, const GroupTab& tab, float* scratch,
                     int max_ranges, void* o_frag) {
    switch (dm.hd) {
        case 32: return launch_attention_hd<32>(st, q, dm, tab, scratch, max_ranges, o_frag);
        case 64: return launch_attention_hd<64>(st, q, dm, tab, scratch, max_ranges, o_frag);
        case 128: return launch_attention_hd<128>(st, q, dm, tab, scratch, max_ranges, o_frag);
    }
    return -1;
}

void launch_out_finish(hipStream_t st, const float* part, int splits, int64_t split_stride,
                       const GroupTab& tab, int d) {
    const size_t n = (size_t)tab.row0[tab.n] * d / 8;
    hipLaunchKernelGGL(out_finish_kernel, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, st, part, splits,
                       split_stride, tab, d);
}

}  // namespace kattn
