// Router backward for up to 128 experts (with fp32 products: 256): the logits' gradient and the gradient of
// the layer's input in one kernel, from the saved probabilities and the fp32 router weights.
//
//   dl[t][e] = p[t][e] (dp[t][e] - sum_i p[t][i] dp[t][i])       (see router_dlogits_kernel)
//   dx[t][k] = m[t][k] sum_e dl[t][e] W_r[k][e] + kept_t dXd[slot_t][k]     (m: input jitter, else 1)
//
// A wave owns 32 tokens and keeps their dl as MFMA fragments in registers: bf16 tokens as two bf16
// terms hi + lo (16 mantissa bits, three products per pair of terms, as the weights), fp32 tokens,
// and bf16 tokens where the expert count is no multiple of 4, as fp32 on the fp32 MFMA (dW_r then
// comes from the fp32 dl too).  The block's four waves walk groups of 64 columns (32 beyond 128
// experts): the group's weights come through registers, one group ahead, are split and laid out
// in LDS in fragment order; the product is turned through LDS so that a wave adds and stores whole
// 128-byte row segments.  Few tokens: several blocks take a column range each and the
// first of them writes dl.
//
// What bounds it: HBM (probabilities, dXd and dx once each: about 50 us at 65536 tokens x 768, 128
// experts) and what two blocks per CU, the most that LDS and registers leave room for, do not
// overlap of products and loads.  Measured (us, before: dlogits + weight split + product kernels):
// 65536 x 768, E 128: 82 (138); 8192: 23 (49); 5003 x 392, E 10 (fp32 products) with the bias sums: 11 (56);
// 65536 with jitter: 97 (160); fp32 256 x 64, E 4: 6 (25), 8192 x 768, E 32: 17 (54).
#include "common.h"
#include "lds_operands.h"
#include "router_wgrad.h"
#include "rows_operands.h"

namespace sw {

struct RouterBwdArgs {
    const float *probs, *dgate, *W_r;
    const int32_t *idx, *counts_g, *tok_slot;
    const void *dXd;
    void *dx;
    float *dlogits;    // dl for dW_r, as that takes it: fp32 [T][E],
    bf16 *dl_split;    // or bf16 terms [T][hi 128 | lo 128], or null
    float *dbr_part;   // [ceil(T / 128)][E] sums of dl, or nullptr
    int T, Tg, d, E, groups_per_block;
    float aux_scale;
    Noise nz;
    int token_blocks;  // of 128 tokens, each once per range of columns, one range after the other;
    int dx_blocks;     // blocks behind these add up the parts of dW_r and db_r
    const float *dWr_part;
    float *dW_r;
    int nsplit;
    DbrArgs db;
};

// EK: 16 experts each.  WIDE: E is a multiple of 4 (rows of E floats are read 16 bytes at a time).
template <typename XT, int EK, bool WIDE>
__global__ __launch_bounds__(256, EK > 8 ? 1 : 2) void router_dx_block_kernel(RouterBwdArgs a) {
    constexpr bool kSplit = sizeof(XT) == 2 && WIDE;            // products of bf16 terms, else fp32
    constexpr int NT = EK > 8 ? 1 : 2, COLS = 32 * NT;          // column tiles and columns of a group
    constexpr int kQuads = COLS * EK * 4 / 256;                 // 4-expert pieces per thread and group
    constexpr int kCPL = 16 / (int)sizeof(XT);                  // columns of a lane's 16-byte piece
    constexpr int kLanesPerRow = COLS / kCPL, kRowsPerPass = 64 / kLanesPerRow, kPasses = 32 / kRowsPerPass;
    constexpr int kPitch = COLS + 4;                            // floats per token of the turn buffer
    typedef XT piece_t __attribute__((ext_vector_type(kCPL)));
    __shared__ __attribute__((aligned(16))) char wlds[NT * EK * 2048];
    __shared__ __attribute__((aligned(16))) float turn_all[4][32 * kPitch];
    if ((int)blockIdx.x >= a.dx_blocks)
        return reduce_partials(a.dWr_part, a.dW_r, (size_t)a.d * a.E, a.nsplit, a.db, blockIdx.x - a.dx_blocks);
    const int range = (int)blockIdx.x / a.token_blocks, tb = (int)blockIdx.x - range * a.token_blocks;
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
    const int half = lane >> 5;
    float *turn = turn_all[wave];
    const int t0 = tb * 128 + wave * 32;
    const int t = t0 + (lane & 31);
    const bool live = t < a.T;
    const int E = a.E;
    const int g_first = range * a.groups_per_block;
    const int g_last = min(g_first + a.groups_per_block, (a.d + COLS - 1) / COLS);

    // ---- the group's weights, one group ahead in registers ----
    f32x4 wreg[kQuads];
    auto load_w = [&](int g) {
#pragma unroll
        for (int i = 0; i < kQuads; ++i) {
            const int at = i * 256 + (int)threadIdx.x;
            const int e = at % (EK * 4) * 4, k = g * COLS + at / (EK * 4);
            const float *src = a.W_r + (size_t)k * E + e;
            f32x4 v = {0.f, 0.f, 0.f, 0.f};
            if (WIDE) {
                if (k < a.d && e < E) v = *(const f32x4 *)src;
            } else {
#pragma unroll
                for (int r = 0; r < 4; ++r)
                    if (k < a.d && e + r < E) v[r] = src[r];
            }
            wreg[i] = v;
        }
    };
    load_w(g_first);

    // ---- dl of the lane's token: experts 16 ks + 8 half .. + 7 ----
    // Loads from places that are there, without a branch around each, so that all are in flight at once; what
    // lies past E or T is replaced by 0 afterwards.  (us with branches / without: 65536 tokens x 768, 128 experts 90 / 82,
    // 8192 29 / 23.  Whole row segments turned in LDS, or eight waves per block that split the next group's weights beside
    // the products: the same.)
    float dl[EK][8];
    const int slot_mine = live ? a.tok_slot[t] : -1;
    {
        const float mean_count = (float)a.Tg / (float)E;
        const int me = live ? a.idx[t] : -1;
        const float dg = live ? a.dgate[t] : 0.f;
        const float *prow = a.probs + (size_t)(live ? t : 0) * E;
        const int32_t *counts = a.counts_g + (size_t)(live ? t / a.Tg : 0) * E;
        float dp[EK][8];
#pragma unroll
        for (int ks = 0; ks < EK; ++ks)
#pragma unroll
            for (int q = 0; q < 2; ++q) {
                const int e0 = ks * 16 + half * 8 + 4 * q;
                if (WIDE) {
                    const int at = min(e0, E - 4);
                    const f32x4 v = *(const f32x4 *)(prow + at);
                    const int4 c = *(const int4 *)(counts + at);
                    const int ci[4] = {c.x, c.y, c.z, c.w};
#pragma unroll
                    for (int r = 0; r < 4; ++r) {
                        dl[ks][4 * q + r] = v[r];
                        dp[ks][4 * q + r] = (float)ci[r];
                    }
                } else {
#pragma unroll
                    for (int r = 0; r < 4; ++r) {
                        const int at = min(e0 + r, E - 1);
                        dl[ks][4 * q + r] = prow[at];
                        dp[ks][4 * q + r] = (float)counts[at];
                    }
                }
            }
        float s = 0.f;
#pragma unroll
        for (int ks = 0; ks < EK; ++ks)
#pragma unroll
            for (int r = 0; r < 8; ++r) {
                const int e = ks * 16 + half * 8 + r;
                // counts centred on their mean: see router_dlogits_kernel
                float v = a.aux_scale * (dp[ks][r] - mean_count);
                if (e == me) v += dg;
                if (!(live && e < E)) dl[ks][r] = 0.f;
                dp[ks][r] = v;
                s += dl[ks][r] * v;
            }
        s += __shfl_xor(s, 32);
#pragma unroll
        for (int ks = 0; ks < EK; ++ks)
#pragma unroll
            for (int r = 0; r < 8; ++r) dl[ks][r] *= dp[ks][r] - s;   // p is 0 past E and past T
    }
    const bool writer = range == 0 && a.nsplit == 0;   // (with parts of dW_r nothing reads dl)
    if (writer && a.dbr_part) {   // column sums over the block's 128 tokens, 16 experts at a time
        __shared__ float dbs[4][EK * 16];
#pragma unroll
        for (int ks = 0; ks < EK; ++ks) {
            float *row = turn + (lane & 31) * 20 + half * 8;
            *(f32x4 *)row = f32x4{dl[ks][0], dl[ks][1], dl[ks][2], dl[ks][3]};
            *(f32x4 *)(row + 4) = f32x4{dl[ks][4], dl[ks][5], dl[ks][6], dl[ks][7]};
            float sum = 0.f;
#pragma unroll
            for (int r = 0; r < 8; ++r) sum += turn[((lane >> 4) * 8 + r) * 20 + (lane & 15)];
            sum += __shfl_xor(sum, 16);
            sum += __shfl_xor(sum, 32);
            if (lane < 16) dbs[wave][ks * 16 + lane] = sum;
        }
        __syncthreads();
        for (int e = threadIdx.x; e < E; e += 256)
            a.dbr_part[(size_t)tb * E + e] = (dbs[0][e] + dbs[1][e]) + (dbs[2][e] + dbs[3][e]);
    }
    bf16x8 hi[EK], lo[EK];
    if (kSplit) {
#pragma unroll
        for (int ks = 0; ks < EK; ++ks)
#pragma unroll
            for (int r = 0; r < 8; ++r) {
                hi[ks][r] = (bf16)dl[ks][r];
                lo[ks][r] = (bf16)(dl[ks][r] - (float)hi[ks][r]);
            }
    }
    if (writer && live) {
        if (kSplit && a.dl_split) {
#pragma unroll
            for (int ks = 0; ks < 8; ++ks) {   // all 128 columns of each half
                bf16 *row = a.dl_split + (size_t)t * 256 + ks * 16 + half * 8;
                const bf16x8 zero = {};
                *(bf16x8 *)row = ks < EK ? hi[ks < EK ? ks : 0] : zero;
                *(bf16x8 *)(row + 128) = ks < EK ? lo[ks < EK ? ks : 0] : zero;
            }
        } else {
#pragma unroll
            for (int ks = 0; ks < EK; ++ks)
#pragma unroll
                for (int q = 0; q < 2; ++q) {
                    const int e0 = ks * 16 + half * 8 + 4 * q;
                    float *out = a.dlogits + (size_t)t * E + e0;
                    if (WIDE) {
                        if (e0 < E)
                            *(f32x4 *)out = f32x4{dl[ks][4 * q], dl[ks][4 * q + 1], dl[ks][4 * q + 2], dl[ks][4 * q + 3]};
                    } else {
#pragma unroll
                        for (int r = 0; r < 4; ++r)
                            if (e0 + r < E) out[r] = dl[ks][4 * q + r];
                    }
                }
        }
    }

    // ---- columns ----
    const int c0 = (lane % kLanesPerRow) * kCPL, r0 = lane / kLanesPerRow;   // of the lane's 16-byte pieces
    const XT *dXd = (const XT *)a.dXd;
    XT *dx = (XT *)a.dx;
    int slot[kPasses];
#pragma unroll
    for (int x = 0; x < kPasses; ++x) slot[x] = __shfl(slot_mine, x * kRowsPerPass + r0);
    // fragment chunk of the lane; rows trade places with (ks, half), so that a wave's writes of
    // one column use all banks
    const uint32_t frag0 = (uint32_t)((half * 32 + ((lane & 31) ^ half)) * 16);
    for (int g = g_first; g < g_last; ++g) {
        __syncthreads();   // the previous group's fragments are read
#pragma unroll
        for (int i = 0; i < kQuads; ++i) {
            const int at = i * 256 + (int)threadIdx.x;
            const int e4 = at % (EK * 4), c = at / (EK * 4);
            const int ks = e4 >> 2, h = (e4 >> 1) & 1, sub = e4 & 1;
            char *frag = wlds + (((c >> 5) * EK + ks) * 2) * 1024 + (h * 32 + ((c & 31) ^ ((ks * 2 + h) & 15))) * 16;
            if (kSplit) {
                bf16x4 whi, wlo;
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    whi[r] = (bf16)wreg[i][r];
                    wlo[r] = (bf16)(wreg[i][r] - (float)whi[r]);
                }
                *(bf16x4 *)(frag + sub * 8) = whi;
                *(bf16x4 *)(frag + 1024 + sub * 8) = wlo;
            } else {
                *(f32x4 *)(frag + sub * 1024) = wreg[i];
            }
        }
        __syncthreads();
        const int col = g * COLS + c0;
        piece_t add[kPasses];
#pragma unroll
        for (int x = 0; x < kPasses; ++x)
            if (slot[x] >= 0 && col < a.d) add[x] = *(const piece_t *)(dXd + (size_t)slot[x] * a.d + col);
        if (g + 1 < g_last) load_w(g + 1);
        f32x16 acc[NT];
#pragma unroll
        for (int n = 0; n < NT; ++n)
#pragma unroll
            for (int r = 0; r < 16; ++r) acc[n][r] = 0.f;
#pragma unroll
        for (int ks = 0; ks < EK; ++ks)
#pragma unroll
            for (int n = 0; n < NT; ++n) {
                const char *frag = wlds + ((n * EK + ks) * 2) * 1024 + (frag0 ^ (uint32_t)(((ks * 2) & 15) << 4));
                if (kSplit) {
                    const bf16x8 whi = *(const bf16x8 *)frag, wlo = *(const bf16x8 *)(frag + 1024);
                    acc[n] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(whi, hi[ks], acc[n], 0, 0, 0);
                    acc[n] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(whi, lo[ks], acc[n], 0, 0, 0);
                    acc[n] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(wlo, hi[ks], acc[n], 0, 0, 0);
                } else {
                    const f32x4 w0 = *(const f32x4 *)frag, w1 = *(const f32x4 *)(frag + 1024);
#pragma unroll
                    for (int r = 0; r < 4; ++r)
                        acc[n] = __builtin_amdgcn_mfma_f32_32x32x2f32(w0[r], dl[ks][r], acc[n], 0, 0, 0);
#pragma unroll
                    for (int r = 0; r < 4; ++r)
                        acc[n] = __builtin_amdgcn_mfma_f32_32x32x2f32(w1[r], dl[ks][4 + r], acc[n], 0, 0, 0);
                }
            }
        // a lane holds, for its token, columns 8 q + 4 half .. + 3 of each tile
#pragma unroll
        for (int n = 0; n < NT; ++n)
#pragma unroll
            for (int q = 0; q < 4; ++q)
                *(f32x4 *)(turn + (lane & 31) * kPitch + n * 32 + q * 8 + half * 4) =
                    f32x4{acc[n][4 * q], acc[n][4 * q + 1], acc[n][4 * q + 2], acc[n][4 * q + 3]};
#pragma unroll
        for (int x = 0; x < kPasses; ++x) {
            const int row = x * kRowsPerPass + r0, tt = t0 + row;
            float v[kCPL];
#pragma unroll
            for (int r = 0; r < kCPL; r += 4) *(f32x4 *)&v[r] = *(const f32x4 *)(turn + row * kPitch + c0 + r);
            if (a.nz.jitter) {
                const uint32_t first = (uint32_t)tt * (uint32_t)a.d + (uint32_t)col;
#pragma unroll
                for (int r = 0; r < kCPL; ++r) v[r] *= jitter_of(a.nz, first + (uint32_t)r);
            }
            piece_t o;
#pragma unroll
            for (int r = 0; r < kCPL; ++r) o[r] = from_f32<XT>(slot[x] >= 0 ? v[r] + to_f32(add[x][r]) : v[r]);
            if (tt < a.T && col < a.d) *(piece_t *)(dx + (size_t)tt * a.d + col) = o;
        }
    }
}

template <typename XT, int EK, bool WIDE>
static void dx_block_launch(RouterBwdArgs a, hipStream_t s) {
    const int groups = (int)ceil_div(a.d, EK > 8 ? 32 : 64), token_blocks = (int)ceil_div(a.T, 128);
    // two blocks per CU want 512 blocks
    const int splits = token_blocks >= 512 ? 1 : (int)ceil_div(512, token_blocks);
    a.groups_per_block = (int)ceil_div(groups, splits < groups ? splits : groups);
    a.token_blocks = token_blocks;
    // (One dimension: the sums' blocks once, not once per range of columns to return at once, two or three per CU at a time for
    // their LDS.  us of a pass, so / here: 64 tokens x 4096, 128 experts 808 / 781, 300 x 8192, 256 fp32 3810 / 3368.)
    a.dx_blocks = token_blocks * (int)ceil_div(groups, a.groups_per_block);
    const int64_t sums = a.nsplit ? ceil_div((int64_t)a.d * a.E, 256) + (a.db.out ? ceil_div(a.E, kDbrExperts) : 0) : 0;
    hipLaunchKernelGGL((router_dx_block_kernel<XT, EK, WIDE>), dim3((unsigned)(a.dx_blocks + sums)), dim3(256), 0, s, a);
}

template <typename XT, int EK> static void dx_block_wide(const RouterBwdArgs &a, hipStream_t s) {
    if (a.E % 4 == 0) dx_block_launch<XT, EK, true>(a, s);
    else dx_block_launch<XT, EK, false>(a, s);
}

// (bf16 terms: at most 128 experts come here)
template <typename XT> static void dx_block_typed(const RouterBwdArgs &a, hipStream_t s) {
    if (a.E <= 32) dx_block_wide<XT, 2>(a, s);
    else if (a.E <= 64) dx_block_wide<XT, 4>(a, s);
    else if (a.E <= 128) dx_block_wide<XT, 8>(a, s);
    else if (sizeof(XT) == 4 && a.E % 4 == 0) dx_block_launch<float, 16, true>(a, s);
    else dx_block_launch<XT, 16, false>(a, s);
}

hipError_t launch_router_dx_block(const Workspace &w, int dtype, float aux_scale, const float *W_r, char *ws,
                                  void *dx, float *dW_r, float *db_r, const RouterWgradArgs &parts, hipStream_t s) {
    ProfScope ps("router_dx", s);
    RouterBwdArgs a{};
    a.probs = (const float *)(ws + w.probs);
    a.dgate = (const float *)(ws + w.dgate);
    a.W_r = W_r;
    a.idx = (const int32_t *)(ws + w.idx);
    a.counts_g = (const int32_t *)(ws + w.counts_g);
    a.tok_slot = (const int32_t *)(ws + w.tok_slot);
    a.dXd = ws + w.dXd;
    a.dx = dx;
    a.dlogits = (float *)(ws + w.dlogits);
    a.dl_split = router_bwd_mfma_supported(w, dtype) ? (bf16 *)(ws + w.dl_split) : nullptr;   // else dl in fp32
    a.dbr_part = db_r && !parts.blocks ? (float *)(ws + w.dbr_part) : nullptr;
    if (parts.blocks) {
        a.dWr_part = parts.part;
        a.dW_r = dW_r;
        a.nsplit = parts.nsplit;
        a.db = DbrArgs{parts.dbr_part, db_r, (int)w.E, parts.nsplit};
    }
    a.T = (int)w.T; a.Tg = (int)w.Tg; a.d = (int)w.d; a.E = (int)w.E;
    a.aux_scale = aux_scale;
    a.nz = w.noise;
    if (dtype == SW_BF16) dx_block_typed<bf16>(a, s);
    else dx_block_typed<float>(a, s);
    return hipGetLastError();
}

}  // namespace sw
