// Router forward for up to 256 experts in one kernel, straight from the fp32 router weights: logits,
// softmax, arg max, gate, in-block ranks and block statistics of 64 or 128 tokens per block.
//
// The router stays an fp32 computation (Sec. 2.4, selective precision).  With bf16 tokens the
// contraction runs on the bf16 matrix cores: a fp32 weight is split, where its fragment is read,
// into three bf16 terms hi + mid + lo (8 + 8 + 8 mantissa bits, the split is exact), so every
// product x * term is exact in fp32 and the MFMA accumulates in fp32.  With fp32 tokens it runs on
// the fp32 MFMA (input jitter applied to the token fragments), and so with bf16 tokens and input jitter, whose x * m is no
// bf16 value (F32P).  Every sum runs over all of d in one
// wave, in order, so a token's logits, and its expert, do not depend on the batch it comes in.
//
// A wave owns one tile of 32 experts and TT / WT MFMA tiles of 32 tokens ("A" = weights, "B" =
// tokens); weights and tokens come through a ring of direct-load stages.  What bounds it: a call of
// few tokens takes one block's chain of loads, splits and MFMAs (64 tokens, d = 768, E = 128: 19 us; the
// 256-token blocks before it and the weight split they needed took 52.  Eight waves that take shares of d
// run in 15, but add up in another order than the blocks of large batches; eight over halves of the tokens
// split every weight twice: 19).  At 65536 tokens it is the
// splits (about 20 vector operations per pair of weights and block) and the token stream together:
// two blocks per CU, one's softmax beside the other's products, 128 tokens per block to halve the
// splits: 57 us (before: 68 plus 5), T = 16384, d = 4096, E = 64: 67 us (before: 210 plus 8).
#include "common.h"
#include "lds_operands.h"
#include "rows_operands.h"

namespace sw {

// One direct load of 4 bytes per lane (see dma16).
__device__ __forceinline__ void dma4(i32x4 rsrc, uint32_t voff, uint32_t soff, uint32_t lds_base) {
    asm volatile("s_mov_b32 m0, %0\n\t"
                 "s_nop 3\n\t"
                 "buffer_load_dword %1, %2, %3 offen lds"
                 :
                 : "s"(lds_base), "v"(voff), "s"(rsrc), "s"(soff)
                 : "memory");
}

// fp32 weights W_r[d][E]: LDS stage [BK k][EP columns].  The half waves of a fragment read are
// 2^SH apart in k (bf16: eight consecutive k each; fp32: odd and even k); columns 32 apart trade places
// where bit SH of k is set, so that they use different banks.  WIDE: 16-byte loads (E a multiple of 4),
// else 4-byte loads.
template <int EP, int BK, int NW, int SH, bool WIDE> struct RouterWeights {
    static constexpr int kLane = WIDE ? 4 : 1;                       // columns per lane and load
    static constexpr int kLoads = BK * EP / (64 * kLane * NW);
    static constexpr int kPerRow = EP / kLane;                       // lanes per k-row
    static constexpr int kRowsPerLoad = kPerRow >= 64 ? 1 : 64 / kPerRow;
    static_assert(kLoads * 64 * kLane * NW == BK * EP, "the stage divides over the waves");
    i32x4 rsrc;
    uint32_t k_step, frag0;

    __device__ __forceinline__ void init(const float *W_r, int d, int E, int lane, int et) {
        rsrc = make_rsrc(W_r, (uint32_t)d * (uint32_t)E * 4u);
        k_step = (uint32_t)E * 4u;
        const int h = lane >> 5;
        const int col = 32 * et + (lane & 31);
        frag0 = (uint32_t)(((h << SH) * EP + (EP >= 64 ? col ^ (h << 5) : col)) * 4);
    }
    __device__ __forceinline__ void issue_one(uint32_t st, int k0, int E, int lane, int wave, int i) const {
        const int at = (wave * kLoads + i) * 64;                     // first lane slot of the load in the stage
        const int kr = at / kPerRow;                                 // its first k-row
        const int kk = kRowsPerLoad > 1 ? lane / kPerRow : 0;
        int col = (kRowsPerLoad > 1 ? lane % kPerRow : lane) * kLane;
        if (EP >= 64) col ^= (((kr + kk) >> SH) & 1) << 5;
        if (kPerRow > 64) col += (at % kPerRow) * kLane;             // a k-row takes several loads
        // columns past E would run into the next k-row: they read zeros instead
        const uint32_t vo = col < E ? (uint32_t)kk * k_step + (uint32_t)col * 4u : kOobOffset;
        const uint32_t so = (uint32_t)(k0 + kr) * k_step;
        const uint32_t dst = st + (uint32_t)at * (4u * kLane);
        if (WIDE) dma16(rsrc, vo, so, dst);
        else dma4(rsrc, vo, so, dst);
    }
    // the lane's N values of the 2 N k of unit u
    template <int N> __device__ __forceinline__ void frag(const char *st, int u, float (&w)[N]) const {
        const char *p = st + frag0 + u * (2 * N * EP * 4);
#pragma unroll
        for (int m = 0; m < N; ++m) w[m] = *(const float *)(p + m * (EP * 4 * (SH == 0 ? 2 : 1)));
    }
};

// ET expert tiles times WT shares of the TT token tiles.
template <typename XT, int ET, int WT, int TT, bool F32P> struct RouterBlock {
    static constexpr int kTok = 32 * TT;
    static constexpr bool kBf16 = sizeof(XT) == 2 && !F32P;   // products
    static constexpr int NW = ET * WT;
    static constexpr int EP = 32 * ET;
    static constexpr int BK = kBf16 && ET <= 2 ? 64 : 32;
    static constexpr int UNIT = kBf16 ? 16 : 8;                   // k of one fragment pair
    static constexpr int kXBytes = kTok * BK * (int)sizeof(XT);
    static constexpr int kStage = kXBytes + BK * EP * 4;
    static constexpr int STAGES = 4 * kStage <= 80 * 1024 || (ET == 8 && kBf16) ? 4 : 3;   // two blocks per CU, but ET = 8
    static constexpr int kPitch = EP + 4;                         // floats per row of the logits tile
    static constexpr int kTile = kTok * kPitch * 4;
    static constexpr int kLds = (STAGES * kStage > kTile ? STAGES * kStage : kTile) + kTok * 4;
    static_assert(kLds <= 160 * 1024, "the block fits a CU");
};

template <typename XT, int ET, int WT, int TT, bool WIDE, bool F32P>
__global__ __launch_bounds__(64 * (RouterBlock<XT, ET, WT, TT, F32P>::NW), 2) void router_block_kernel(
    const XT *__restrict__ x, const float *__restrict__ W_r, const float *__restrict__ b_r,
    float *__restrict__ probs, float *__restrict__ logits_out, int32_t *__restrict__ idx_out,
    float *__restrict__ gate_out, int32_t *__restrict__ idx_ws, float *__restrict__ gate_ws,
    int32_t *__restrict__ local_rank, int32_t *__restrict__ block_counts,
    float *__restrict__ block_psum, int nbg, int Tg, int d, int E, Noise nz) {
    typedef RouterBlock<XT, ET, WT, TT, F32P> R;
    constexpr bool BF = R::kBf16;
    constexpr int NW = R::NW, EP = R::EP, BK = R::BK, STAGES = R::STAGES, TOK = R::kTok;
    constexpr int TW = TT / WT, NX = NW < 4 ? NW : 4;   // token tiles per wave, waves that load tokens
    extern __shared__ __attribute__((aligned(16))) char lds[];
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int et = wave % ET, wt = wave / ET;
    const uint32_t lds0 = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) char *)lds;
    const int b = blockIdx.x;
    int t0, tend;   // the block's tokens, inside one routing group
    block_token_range(b, nbg, Tg, TOK, t0, tend);

    typename std::conditional<sizeof(XT) == 2, RowsDirect<TOK, NX, BK>, F32Direct<TOK, NX>>::type ox;
    RouterWeights<EP, BK, NW, BF ? 3 : 0, WIDE> ow;
    ox.init(x, d, t0, tend, d, lane, wave % NX);   // (waves past the fourth repeat the loads of the first four)
    ox.init_frag(lane, wt * TW * 32);
    ow.init(W_r, d, E, lane, et);
    constexpr int kLX = decltype(ox)::kLoads, kLoads = kLX + decltype(ow)::kLoads;
    const int nk = (d + BK - 1) / BK;
    auto issue = [&](int kt) {   // (steps past the end: never read)
        const uint32_t st = lds0 + (uint32_t)((kt % STAGES) * R::kStage);
#pragma unroll
        for (int i = 0; i < kLX; ++i) ox.issue_one(st, kt * BK, wave % NX, i);
#pragma unroll
        for (int i = 0; i < decltype(ow)::kLoads; ++i) ow.issue_one(st + R::kXBytes, kt * BK, E, lane, wave, i);
    };

    f32x16 acc[TW];
#pragma unroll
    for (int tt = 0; tt < TW; ++tt)
#pragma unroll
        for (int r = 0; r < 16; ++r) acc[tt][r] = 0.f;

#pragma unroll
    for (int s = 0; s < STAGES - 1; ++s) issue(s);
    for (int kt = 0; kt < nk; ++kt) {
        rows_wait_vmcnt<(STAGES - 2) * kLoads>();
        __syncthreads();
        issue(kt + STAGES - 1);
        const char *sx = lds + (kt % STAGES) * R::kStage, *sw_ = sx + R::kXBytes;
#pragma unroll
        for (int u = 0; u < BK / R::UNIT; ++u) {
            if constexpr (BF) {
                float w[8];
                ow.template frag<8>(sw_, u, w);
                bf16x8 fx[TW];
                uint32_t term[3][4];
#pragma unroll
                for (int tt = 0; tt < TW; ++tt) fx[tt] = ox.frag(sx, tt, u);
#pragma unroll
                for (int m = 0; m < 4; ++m) {   // a pair at a time: one conversion instruction per term
                    float a = w[2 * m], c = w[2 * m + 1];
#pragma unroll
                    for (int s = 0; s < 3; ++s) {
                        const uint32_t pr = pack_bf16(a, c);
                        term[s][m] = pr;
                        a -= __uint_as_float(pr << 16);
                        c -= __uint_as_float(pr & 0xffff0000u);
                    }
                }
#pragma unroll
                for (int s = 0; s < 3; ++s)
#pragma unroll
                    for (int tt = 0; tt < TW; ++tt)
                        acc[tt] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(
                            __builtin_bit_cast(bf16x8, u32x4{term[s][0], term[s][1], term[s][2], term[s][3]}), fx[tt],
                            acc[tt], 0, 0, 0);
            } else {
                float w[4];
                ow.template frag<4>(sw_, u, w);
                f32x4 fx[TW];
#pragma unroll
                for (int tt = 0; tt < TW; ++tt) {
                    if constexpr (F32P) {   // the lane's four (every other) of the token's eight bf16 values
                        const u32x4 v = *(const u32x4 *)(sx + ((ox.frag0 ^ (uint32_t)((lane >> 5) << 4) ^ (uint32_t)(u << 4)) +
                                                               (uint32_t)(tt * 32 * 2 * BK)));
#pragma unroll
                        for (int m = 0; m < 4; ++m) fx[tt][m] = __uint_as_float(lane >> 5 ? v[m] & 0xffff0000u : v[m] << 16);
                    } else {
                        fx[tt] = ox.frag4(sx, tt, u);
                    }
                    if (nz.jitter) {   // input jitter (App. C): the router sees x * m
                        const uint32_t t = (uint32_t)(t0 + (wt * TW + tt) * 32 + (lane & 31));
                        const uint32_t at = t * (uint32_t)d + (uint32_t)(kt * BK + u * 8 + (lane >> 5));
#pragma unroll
                        for (int m = 0; m < 4; ++m) fx[tt][m] *= jitter_of(nz, at + 2u * (uint32_t)m);
                    }
                }
#pragma unroll
                for (int m = 0; m < 4; ++m)
#pragma unroll
                    for (int tt = 0; tt < TW; ++tt)
                        acc[tt] = __builtin_amdgcn_mfma_f32_32x32x2f32(w[m], fx[tt][m], acc[tt], 0, 0, 0);
            }
        }
    }
    rows_wait_vmcnt<0>();
    __syncthreads();

    // ---- logits into LDS, [tokens][EP] ----------------------------------------
    float *tile = (float *)lds;
    int32_t *idx_s = (int32_t *)(lds + R::kLds - TOK * 4);
#pragma unroll
    for (int tt = 0; tt < TW; ++tt)
#pragma unroll
        for (int g = 0; g < 4; ++g)
            *(float4 *)(tile + ((wt * TW + tt) * 32 + (lane & 31)) * R::kPitch + et * 32 + 8 * g + 4 * (lane >> 5)) =
                make_float4(acc[tt][4 * g], acc[tt][4 * g + 1], acc[tt][4 * g + 2], acc[tt][4 * g + 3]);
    __syncthreads();

    // ---- softmax, arg max, gate: LT lanes share a token, lane l takes chunks l, l + LT, .. of four experts
    constexpr int LT = 64 * NW / TOK;
    const int row = tid / LT, l = tid % LT;
    const int t = t0 + row;
    constexpr int kJ = EP / 4 / LT;
    float4 h[kJ];
    float best = -INFINITY;
    int besti = 0x7fffffff;
#pragma unroll
    for (int j = 0; j < kJ; ++j) {
        const int e = 4 * (j * LT + l);
        float4 v = *(const float4 *)(tile + row * R::kPitch + e);
        float *hv = (float *)&v;
#pragma unroll
        for (int m = 0; m < 4; ++m) {
            hv[m] = e + m < E ? hv[m] + (b_r ? b_r[e + m] : 0.f) : -INFINITY;
            if (hv[m] > best) { best = hv[m]; besti = e + m; }   // ascending: lowest index kept on ties
        }
        h[j] = v;
    }
    auto put = [&](float *rowp, int e, const float4 &v) {   // four experts of a [T][E] row
        if ((E & 3) == 0) {
            if (e < E) *(float4 *)(rowp + e) = v;
        } else {
            const float *hv = (const float *)&v;
#pragma unroll
            for (int m = 0; m < 4; ++m)
                if (e + m < E) rowp[e + m] = hv[m];
        }
    };
    if (logits_out && t < tend)
#pragma unroll
        for (int j = 0; j < kJ; ++j) put(logits_out + (size_t)t * E, 4 * (j * LT + l), h[j]);
#pragma unroll
    for (int m = 1; m < LT; m <<= 1) {
        const float ov = __shfl_xor(best, m, kWave);
        const int oi = __shfl_xor(besti, m, kWave);
        if (ov > best || (ov == best && oi < besti)) { best = ov; besti = oi; }
    }
    float z = 0.f;
#pragma unroll
    for (int j = 0; j < kJ; ++j) {
        float *hv = (float *)&h[j];
#pragma unroll
        for (int m = 0; m < 4; ++m) {
            // exp(-inf) = 0 for absent experts; the hardware exp2 is accurate to about one ulp,
            // the scaled argument adds |h - best| 2^-24: far inside the 1e-5 budget
            hv[m] = __expf(hv[m] - best);
            z += hv[m];
        }
    }
#pragma unroll
    for (int m = 1; m < LT; m <<= 1) z += __shfl_xor(z, m, kWave);
    const float rz = 1.0f / z;   // exp(0) / z: also the probability of the arg max
#pragma unroll
    for (int j = 0; j < kJ; ++j) {
        const int e = 4 * (j * LT + l);
        float4 p = h[j];
        p.x *= rz; p.y *= rz; p.z *= rz; p.w *= rz;
        if (t >= tend) p = make_float4(0.f, 0.f, 0.f, 0.f);
        *(float4 *)(tile + row * R::kPitch + e) = p;   // (the lane's own chunks: nobody else reads them)
        if (t < tend) put(probs + (size_t)t * E, e, p);
    }
    if (l == 0) {
        if (besti >= E) besti = 0;   // (no logit above -inf, not even one that is no NaN: the lowest index)
        idx_s[row] = t < tend ? besti : -1;
        if (t < tend) {
            idx_out[t] = besti;
            idx_ws[t] = besti;
            gate_out[t] = rz;
            gate_ws[t] = rz;
        }
    }
    __syncthreads();

    // ---- block statistics ---------------------------------------------------------------
    // rank of each token among the block's earlier tokens of the same expert: the last waves,
    // which have no columns to sum when E <= 128, take 64 tokens each
    if (wave >= NW - TOK / 64) {
        const int first = 64 * (wave - (NW - TOK / 64));
        const int me = idx_s[first + lane];
        int r = 0;
        for (int q = 0; q < first; ++q) r += idx_s[q] == me ? 1 : 0;
#pragma unroll
        for (int sl = 0; sl < 64; ++sl) {
            const int other = __builtin_amdgcn_readlane(me, sl);
            r += (sl < lane && other == me) ? 1 : 0;
        }
        if (me >= 0) local_rank[t0 + first + lane] = r;
    }
    for (int e = tid; e < E; e += 64 * NW) {
        // column sums in a fixed order: four interleaved chains, then ((s0 + s1) + (s2 + s3))
        float s[4] = {0.f, 0.f, 0.f, 0.f};
        int n = 0;
#pragma unroll 4
        for (int q = 0; q < TOK; q += 4)
#pragma unroll
            for (int m = 0; m < 4; ++m) {
                s[m] += tile[(q + m) * R::kPitch + e];   // 0 for tokens past the end
                n += idx_s[q + m] == e ? 1 : 0;
            }
        block_psum[(size_t)b * E + e] = (s[0] + s[1]) + (s[2] + s[3]);
        block_counts[(size_t)b * E + e] = n;
    }
}

// Up to 256 experts whose weights and tokens fit a buffer descriptor each.  Input jitter on bf16 tokens, for large layers
// with a multiple of 4 experts: planes of x * m (router_mfma.hip), whose products are cheaper, but which take three launches
// and long chains of few blocks.  us of a pass (d_ff 256 unless said), planes or vector ALUs / here:
//   experts without 4 as a divisor: 32 x 2400, 10 experts 1223 / 518
//   up to 64: 8192 x 2048, 32 experts 510 / 353, 32768 x 1024 x 2048, 32 experts 1156 / 1067, 65536 x 768 x 512, 64 experts 846 / 818
//   up to 128, up to 16384 tokens (a block per CU) and 1e9 products: 512 x 768 x 1024, 128 experts 528 / 500, 10000 x 768 x 3072,
//     128 experts 984 / 968; 16384 x 768 x 3072, 128 experts 1099 / 1104, 17000 x 128, 128 experts 154 / 171, 65536 x 768 x 3072,
//     128 experts 2426 / 2753
//   up to 256, short rows and few products: 4000 x 256, 256 experts 186 / 162; 2048 x 768, 256 experts 336 / 343, 8000 x 256, 256
//     experts 198 / 208, 64 x 2048, 256 experts 475 / 497 (a block reads and splits all of W_r, however few its tokens)
// Tokens per block: 128 halves what the weights cost (traffic and splits) once there are blocks
// for two per CU.
int router_block_tokens(const switch_config *cfg) {
    return cfg->act_dtype == SW_BF16 && cfg->jitter_eps == 0.f && cfg->E <= 128 && cfg->T >= 32768 ? 128 : 64;
}

static bool jitter_takes_planes(const switch_config *cfg) {
    const double products = (double)cfg->T * (double)cfg->d_model * (double)cfg->E;
    if (cfg->act_dtype != SW_BF16 || !(cfg->jitter_eps > 0.f) || cfg->E % 4 != 0) return false;
    if (cfg->E <= 64) return false;
    if (cfg->E <= 128) return products > 1e9 || cfg->T > 16384;
    return products > 3e8 || cfg->d_model > 1024;
}

bool router_block_supported(const switch_config *cfg) {
    const double elt = cfg->act_dtype == SW_BF16 ? 2. : 4.;
    return cfg->E <= 256 && (double)cfg->d_model * (double)cfg->E * 4. < 2147483647. &&
           (double)cfg->T * (double)cfg->d_model * elt < 2147483647. && !jitter_takes_planes(cfg);
}

template <typename XT, int ET, int WT, int TT, bool WIDE, bool F32P>
static hipError_t router_block_launch(const Workspace &w, const void *x, const float *W_r, const float *b_r,
                                      char *ws, int32_t *expert_index, float *gate, float *router_logits,
                                      hipStream_t s) {
    auto kern = router_block_kernel<XT, ET, WT, TT, WIDE, F32P>;
    typedef RouterBlock<XT, ET, WT, TT, F32P> R;
    static PerDeviceOnce once;
    hipError_t err = once_per_device(once, [&] {
        return hipFuncSetAttribute((const void *)kern, hipFuncAttributeMaxDynamicSharedMemorySize, R::kLds);
    });
    if (err != hipSuccess) return err;
    hipLaunchKernelGGL(kern, dim3((unsigned)w.nb), dim3(64 * R::NW), R::kLds, s, (const XT *)x, W_r, b_r,
                       (float *)(ws + w.probs), router_logits, expert_index, gate, (int32_t *)(ws + w.idx),
                       (float *)(ws + w.gate), (int32_t *)(ws + w.local_rank),
                       (int32_t *)(ws + w.block_counts), (float *)(ws + w.block_psum), (int)w.nbg,
                       (int)w.Tg, (int)w.d, (int)w.E, w.noise);
    return hipGetLastError();
}

template <typename XT, bool F32P>
static hipError_t router_block_typed(const Workspace &w, const void *x, const float *W_r, const float *b_r,
                                     char *ws, int32_t *expert_index, float *gate, float *logits, hipStream_t s) {
#define SW_RB(ET, WT, TT)                                                                                          \
    (w.E % 4 == 0 ? router_block_launch<XT, ET, WT, TT, true, F32P>(w, x, W_r, b_r, ws, expert_index, gate, logits, s) \
                  : router_block_launch<XT, ET, WT, TT, false, F32P>(w, x, W_r, b_r, ws, expert_index, gate, logits, s))
    if constexpr (sizeof(XT) == 2 && !F32P)
        if (w.tb == 128) return w.E <= 32 ? SW_RB(1, 4, 4) : w.E <= 64 ? SW_RB(2, 2, 4) : SW_RB(4, 1, 4);
    if (w.E <= 32) return SW_RB(1, 2, 2);
    if (w.E <= 64) return SW_RB(2, 2, 2);
    return w.E <= 128 ? SW_RB(4, 1, 2) : SW_RB(8, 1, 2);
#undef SW_RB
}

hipError_t launch_router_block(const Workspace &w, int dtype, const void *x, const float *W_r,
                               const float *b_r, char *ws, int32_t *expert_index, float *gate,
                               float *router_logits, hipStream_t s) {
    ProfScope ps("router_fwd", s);
    if (dtype != SW_BF16)
        return router_block_typed<float, false>(w, x, W_r, b_r, ws, expert_index, gate, router_logits, s);
    return w.noise.jitter ? router_block_typed<bf16, true>(w, x, W_r, b_r, ws, expert_index, gate, router_logits, s)
                          : router_block_typed<bf16, false>(w, x, W_r, b_r, ws, expert_index, gate, router_logits, s);
}

}  // namespace sw
