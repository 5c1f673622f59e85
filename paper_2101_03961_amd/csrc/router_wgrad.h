// Gradient of the router's weights beside other work: its parts in blocks of the launch that computes the experts'
// weight gradients, their sums in blocks of the launch that computes dx.
//
//   dW_r[k][j] = sum_t m[t][k] x[t][k] dl[t][j],   dl[t][j] = p[t][j] (dp[t][j] - s[t]),   db_r[j] = sum_t dl[t][j]
//
// (m: input jitter, else 1; dp: see router_dlogits_kernel.)  dl is made here, from the probabilities and
// s[t] = sum_i p[t][i] dp[t][i], which the combine's backward pass leaves per token, so neither part waits for the
// kernel that computes dx or needs memory for dl.  Products and sums in fp32.  What bounds it as launches of its own:
// two more steps in a chain of a dozen, a few microseconds each (router_wgrad_splits says where it pays).
#pragma once
#include "common.h"

namespace sw {

// db_r[e] = sum over parts of part[q][e], in blocks behind those of a dW_r reduction: kDbrExperts
// experts per block, eight interleaved chains per expert, added in order.
constexpr int kDbrExperts = 32;
struct DbrArgs {
    const float *part;   // [nparts][E]
    float *out;          // nullptr: no bias
    int E, nparts;
};
__device__ static void reduce_dbr(const DbrArgs &a, int block) {
    __shared__ float sums[8][kDbrExperts];
    const int j = threadIdx.x % kDbrExperts, chain = threadIdx.x / kDbrExperts;
    const int e = block * kDbrExperts + j;
    float s = 0.f;
    if (e < a.E) {
#pragma unroll 8
        for (int q = chain; q < a.nparts; q += 8) s += a.part[(size_t)q * a.E + e];
    }
    sums[chain][j] = s;
    __syncthreads();
    if (chain != 0 || e >= a.E) return;
    for (int c = 1; c < 8; ++c) s += sums[c][j];
    a.out[e] = s;
}

// out[i] = sum over splits of part[q][i], fixed order; then db_r
__device__ __forceinline__ void reduce_partials(const float *part, float *out, size_t n, int nsplit, const DbrArgs &db,
                                                size_t block) {
    const size_t blocks = (n + 255) / 256;
    if (block >= blocks) return reduce_dbr(db, (int)(block - blocks));
    const size_t i = block * 256 + threadIdx.x;
    if (i >= n) return;
    // (32 loads in flight, then eight: a small matrix is one block with a chain of up to 256 parts.  us of the launch that
    // computes dx, eight / here: 36737 tokens of 40, 5 experts, 250 parts 16 / 10)
    float s = 0.f;
    int q = 0;
    for (; q + 32 <= nsplit; q += 32) {
        float v[32];
#pragma unroll
        for (int u = 0; u < 32; ++u) v[u] = part[(size_t)(q + u) * n + i];
#pragma unroll
        for (int u = 0; u < 32; ++u) s += v[u];
    }
#pragma unroll 8
    for (; q < nsplit; ++q) s += part[(size_t)q * n + i];
    out[i] = s;
}

struct RouterWgradArgs {
    int blocks;              // 0: none
    const void *x;
    const float *probs, *dgate, *rowsum;
    const int32_t *idx, *counts_g;
    float *part;             // [nsplit][d][E]
    float *dbr_part;         // [nsplit][E], or null
    int T, Tg, d, E, nsplit, tokens_per_split, tiles_k;
    float aux_scale;
    Noise nz;
};

// Tile of 4096 elements, as many experts as there are up to 64 (a multiple of 16), by as many k; tokens at a time.
inline int router_wgrad_experts(int64_t E) { return E <= 16 ? 16 : E <= 32 ? 32 : 64; }
constexpr int kRwElements = 4096, kRwTokens = 32;
constexpr int kRwLds = 32 * (128 + 4 + 32 + 4) * 4;   // (the largest)

// Block of 256 threads: KT k x JT experts over one range of tokens, TOK at a time, the next TOK in registers.
// Thread: 4 k x 4 experts.  A chain of sums takes kRwChain tokens: where memory allows few parts, a part has
// thousands (error against 64 bits, one chain per part / here: 30000 tokens of 4096, 256 experts, 3 parts 1.7e-6 / 3.0e-7; 20000
// of 1024, 15 parts 6.4e-7 / 2.4e-7; same time).
constexpr int kRwChain = 128;
template <typename XT, int JT> __device__ __forceinline__ void router_wgrad_tile(const RouterWgradArgs &a, int block, char *lds) {
    constexpr int KT = kRwElements / JT, TOK = JT == 16 ? 16 : 32;
    constexpr int kRowsX = 1024 / KT, kPassX = TOK / kRowsX, kRowsL = 1024 / JT, kPassL = (TOK + kRowsL - 1) / kRowsL;
    constexpr int kPitchX = KT + 4, kPitchL = JT + 4;
    static_assert(TOK * (kPitchX + kPitchL) * 4 <= kRwLds, "");
    typedef XT x4 __attribute__((ext_vector_type(4)));
    typedef float f4 __attribute__((ext_vector_type(4)));
    float *xs = (float *)lds, *ls = xs + TOK * kPitchX;
    const int split = block % a.nsplit, tile = block / a.nsplit;
    const int k0 = tile % a.tiles_k * KT, j0 = tile / a.tiles_k * JT;
    const int t_lo = split * a.tokens_per_split, t_hi = min(t_lo + a.tokens_per_split, a.T);
    const int tid = threadIdx.x;
    const int xrow = tid / (KT / 4), xcol = tid % (KT / 4) * 4, lrow = tid / (JT / 4), lcol = tid % (JT / 4) * 4;
    const float mean_count = (float)a.Tg / (float)a.E;
    // as they lie in memory: what is made of them waits for them, and is made behind the products
    x4 xr[kPassX];
    float pr[kPassL][4], dgr[kPassL], sr[kPassL];
    int cr[kPassL][4], mer[kPassL];
    auto load = [&](int t0) {
#pragma unroll
        for (int h = 0; h < kPassX; ++h) {
            const int t = t0 + xrow + kRowsX * h;
            xr[h] = x4{};
            if (t < t_hi && k0 + xcol < a.d)   // d is a multiple of 4
                xr[h] = *(const x4 *)((const XT *)a.x + (size_t)t * a.d + k0 + xcol);
        }
#pragma unroll
        for (int h = 0; h < kPassL; ++h) {
            const int row = lrow + kRowsL * h, t = t0 + row;
            const bool in = row < TOK && t < t_hi;
            mer[h] = in ? a.idx[t] : -1;
            dgr[h] = in ? a.dgate[t] : 0.f;
            sr[h] = in ? a.rowsum[t] : 0.f;
            const int32_t *counts = a.counts_g + (size_t)(in ? t / a.Tg : 0) * a.E;
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                const int e = j0 + lcol + u;
                cr[h][u] = e < a.E ? counts[e] : 0;
                pr[h][u] = in && e < a.E ? a.probs[(size_t)t * a.E + e] : 0.f;
            }
        }
    };
    auto put = [&](int t0) {
#pragma unroll
        for (int h = 0; h < kPassX; ++h) {
            const int row = xrow + kRowsX * h;
            f4 v;
#pragma unroll
            for (int u = 0; u < 4; ++u) v[u] = to_f32((XT)xr[h][u]);
            if (a.nz.jitter)
#pragma unroll
                for (int u = 0; u < 4; ++u)
                    v[u] *= jitter_of(a.nz, (uint32_t)(t0 + row) * (uint32_t)a.d + (uint32_t)(k0 + xcol + u));
            *(f4 *)(xs + row * kPitchX + xcol) = v;
        }
#pragma unroll
        for (int h = 0; h < kPassL; ++h) {
            const int row = lrow + kRowsL * h;
            if (row >= TOK) continue;
            f4 v;
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                float dp = a.aux_scale * ((float)cr[h][u] - mean_count);
                if (j0 + lcol + u == mer[h]) dp += dgr[h];
                v[u] = pr[h][u] * (dp - sr[h]);   // (0 past the experts and the tokens)
            }
            *(f4 *)(ls + row * kPitchL + lcol) = v;
        }
    };
    const int tx = lcol, ty = lrow * 4;
    float acc[4][4] = {}, total[4][4] = {};
    float db = 0.f;
    const bool bias = a.dbr_part && k0 == 0 && tid < JT;
    load(t_lo);
    for (int t0 = t_lo; t0 < t_hi; t0 += TOK) {
        __syncthreads();   // the tokens before are used
        put(t0);
        __syncthreads();
        if (t0 + TOK < t_hi) load(t0 + TOK);
#pragma unroll 8
        for (int t = 0; t < TOK; ++t) {
            const f4 xv = *(const f4 *)(xs + t * kPitchX + ty), lv = *(const f4 *)(ls + t * kPitchL + tx);
#pragma unroll
            for (int i = 0; i < 4; ++i)
#pragma unroll
                for (int j = 0; j < 4; ++j) acc[i][j] = fmaf(xv[i], lv[j], acc[i][j]);
        }
        if (bias) {
            float s = 0.f;
#pragma unroll 8
            for (int t = 0; t < TOK; ++t) s += ls[t * kPitchL + tid];
            db += s;
        }
        if ((t0 - t_lo) % kRwChain == kRwChain - TOK || t0 + TOK >= t_hi)
#pragma unroll
            for (int i = 0; i < 4; ++i)
#pragma unroll
                for (int j = 0; j < 4; ++j) {
                    total[i][j] += acc[i][j];
                    acc[i][j] = 0.f;
                }
    }
    float *out = a.part + (size_t)split * a.d * a.E;
#pragma unroll
    for (int i = 0; i < 4; ++i)
        if (k0 + ty + i < a.d)
#pragma unroll
            for (int j = 0; j < 4; ++j)
                if (j0 + tx + j < a.E) out[(size_t)(k0 + ty + i) * a.E + j0 + tx + j] = total[i][j];
    if (bias && j0 + tid < a.E) a.dbr_part[(size_t)split * a.E + j0 + tid] = db;
}

template <typename XT> __device__ __forceinline__ void router_wgrad_block(const RouterWgradArgs &a, int block, char *lds) {
    if (a.E <= 16) router_wgrad_tile<XT, 16>(a, block, lds);
    else if (a.E <= 32) router_wgrad_tile<XT, 32>(a, block, lds);
    else router_wgrad_tile<XT, 64>(a, block, lds);
}

}  // namespace sw
