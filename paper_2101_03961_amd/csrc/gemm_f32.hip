// Grouped expert GEMMs for the all-fp32 configuration (act_dtype = SW_F32): fp32 products and
// sums on the matrix cores (v_mfma_f32_32x32x2_f32, 157 TFLOP/s), and a plain FMA kernel with 64-bit
// addresses for layers whose per-expert matrices reach 2 GB or whose tiles fill more than one grid dimension.
#include <math.h>

#include "common.h"
#include "lds_operands.h"
#include "router_wgrad.h"
#include "rows_operands.h"

namespace sw {

struct GemmF32Args {
    const float *Q;      // Q_e(q,k) = Q[e*q_batch + q*q_rs + k*q_ks]
    const float *P;      // P_e(p,k) = P[e*p_batch + p*p_rs + k*p_ks]
    float *Cout;         // C_e[q][p] = Cout[e*c_batch + q*ldc + p]
    const float *mask;   // same layout as Cout, or nullptr
    size_t q_batch, p_batch, c_batch;
    long q_rs, q_ks, p_rs, p_ks, ldc;
    int Qdim, Pdim, Kdim;
    const int32_t *kept;
    int q_limited;       // rows q >= kept[e] are not computed / stored
    int k_limited;       // reduction runs over k < kept[e]
    int epi;             // 0 none, 1 ReLU (+ expert dropout), 2 multiply by [mask > 0] (and by
                         // the dropout scale of the surviving units)
    const int32_t *slot_token;   // epi 1 with dropout, F32_COMBINE: token of slot e * slots + q
    const float *slot_gate;      // F32_COMBINE: its gate, and the output rows by token
    float *y;
    long slots;
    Noise nz;
};

constexpr int kF32Tile = 64;
constexpr int kF32KC = 16;
constexpr int kF32Flush = 256;   // products per chain of the two-level sum

__global__ __launch_bounds__(256) void gemm_f32_kernel(GemmF32Args a) {
    __shared__ float qs[kF32KC][kF32Tile + 4];
    __shared__ float ps[kF32KC][kF32Tile + 4];
    const int e = blockIdx.z;
    const int q0 = blockIdx.y * kF32Tile;
    const int p0 = blockIdx.x * kF32Tile;
    const int lim = a.kept[e];
    const int qlim = a.q_limited ? (lim < a.Qdim ? lim : a.Qdim) : a.Qdim;
    const int klim = a.k_limited ? (lim < a.Kdim ? lim : a.Kdim) : a.Kdim;
    if (q0 >= qlim) return;
    const float *Q = a.Q + (size_t)e * a.q_batch;
    const float *P = a.P + (size_t)e * a.p_batch;
    const int tid = threadIdx.x;
    const int tx = tid % 16, ty = tid / 16;
    // Two-level sums: a running chain of at most kF32Flush products is folded into a total, so
    // that the rounding error of a long reduction (thousands of slots in a weight gradient)
    // grows with the square roots of the two lengths instead of with the whole length.
    float acc[4][4], total[4][4];
#pragma unroll
    for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int j = 0; j < 4; ++j) acc[i][j] = total[i][j] = 0.f;
    for (int k0 = 0; k0 < klim; k0 += kF32KC) {
        if (k0 != 0 && k0 % kF32Flush == 0) {
#pragma unroll
            for (int i = 0; i < 4; ++i)
#pragma unroll
                for (int j = 0; j < 4; ++j) {
                    total[i][j] += acc[i][j];
                    acc[i][j] = 0.f;
                }
        }
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const int id = tid + i * 256;
            int r, kk;
            // pick the faster-varying index to be the contiguous one in memory
            if (a.q_ks == 1) { kk = id % kF32KC; r = id / kF32KC; } else { r = id % kF32Tile; kk = id / kF32Tile; }
            float v = 0.f;
            if (q0 + r < qlim && k0 + kk < klim) v = Q[(long)(q0 + r) * a.q_rs + (long)(k0 + kk) * a.q_ks];
            qs[kk][r] = v;
            if (a.p_ks == 1) { kk = id % kF32KC; r = id / kF32KC; } else { r = id % kF32Tile; kk = id / kF32Tile; }
            v = 0.f;
            if (p0 + r < a.Pdim && k0 + kk < klim) v = P[(long)(p0 + r) * a.p_rs + (long)(k0 + kk) * a.p_ks];
            ps[kk][r] = v;
        }
        __syncthreads();
#pragma unroll
        for (int kk = 0; kk < kF32KC; ++kk) {
            float qv[4], pv[4];
#pragma unroll
            for (int i = 0; i < 4; ++i) qv[i] = qs[kk][ty * 4 + i];
#pragma unroll
            for (int j = 0; j < 4; ++j) pv[j] = ps[kk][tx * 4 + j];
#pragma unroll
            for (int i = 0; i < 4; ++i)
#pragma unroll
                for (int j = 0; j < 4; ++j) acc[i][j] = fmaf(qv[i], pv[j], acc[i][j]);
        }
        __syncthreads();
    }
    float *Cout = a.Cout + (size_t)e * a.c_batch;
    const float *mask = a.mask ? a.mask + (size_t)e * a.c_batch : nullptr;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        const int q = q0 + ty * 4 + i;
        if (q >= qlim) continue;
        uint32_t row_idx = 0;   // index of the token's first hidden unit in the dropout stream
        if (a.epi == 1 && a.nz.dropout)
            row_idx = (uint32_t)a.slot_token[(size_t)e * a.slots + q] * (uint32_t)a.Pdim;
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const int p = p0 + tx * 4 + j;
            if (p >= a.Pdim) continue;
            float v = total[i][j] + acc[i][j];
            if (a.epi == 1) {
                v = v > 0.f ? v : 0.f;
                if (a.nz.dropout)   // Sec. 2.4: expert dropout on the hidden activation
                    v = dropout_keeps(a.nz, row_idx + (uint32_t)p) ? v * a.nz.drop_scale : 0.f;
            }
            // a unit passes the gradient iff it was active and survived dropout
            if (a.epi == 2) v = mask[(long)q * a.ldc + p] > 0.f ? v * a.nz.drop_scale : 0.f;
            Cout[(long)q * a.ldc + p] = v;
        }
    }
}

// ---- fp32 on the matrix cores -----------------------------------------------------------
// One tile per block, QB x PB, WP x WQ waves of IP x IQ MFMA tiles of S x S (32x32x2 or 16x16x4); k advances
// 32 at a time through STAGES LDS stages filled by direct loads.  Bound by the MFMA rate (64 cycles for
// 4096 FLOP per SIMD, of either shape): a 64 x 64 step takes 1024 cycles and needs 16 KB, so operand traffic is no issue
// and the tile is chosen small enough to fill the chip; waves whose rows do not exist skip their
// MFMAs.  Measured (32 experts x 256 tokens x 768 x 3072, us per launch): 345-392 = 98-111 TFLOP/s,
// the FMA kernel 827-1269.
// Two-level sums as in the FMA kernel: chains of kF32Flush products are folded into a total.
//
// k runs in order: an MFMA of S x S multiplies the next 64 / S of them one after the other, so that every
// sum is the same chain of fused multiply-adds as the FMA kernel's, bit for bit, with each tile.
// [k][row] operand: LDS [32 k][R]; rows S apart trade places in odd k-rows (S = 16: in k-rows 4 n + 2 and
// 4 n + 3), so that the k-rows of a read use different banks.
template <int R, int NW, int S> struct F32Trans {
    static_assert(S == 32 ? R > 32 : R == 32, "rows S apart, whose k-rows would meet in a bank");
    static __device__ __forceinline__ int turn(int k) { return S == 32 ? (k & 1) << 5 : (k >> 1 & 1) << 4; }
    static constexpr int kLoads = R * 32 * 4 / (1024 * NW);
    static constexpr int kChunks = R / 4;              // 16-byte chunks of a k-row
    static constexpr int kRowsPerLoad = 64 / kChunks;  // k-rows of one wave-wide load
    static_assert(kLoads * NW * kRowsPerLoad == 32 && kRowsPerLoad % (64 / S) == 0, "k-rows divide over the waves");
    i32x4 rsrc;
    uint32_t voff, k_step, frag0;
    __device__ __forceinline__ void init(const float *base, int ld, int row0, int rowlim, int klim,
                                         int lane, int wave) {
        rsrc = make_rsrc(base, (uint32_t)klim * (uint32_t)ld * 4u);
        k_step = (uint32_t)ld * 4u;
        const int kk = lane / kChunks;
        const int row = row0 + ((lane % kChunks) ^ (turn(kk) >> 2)) * 4;
        voff = row < rowlim ? ((uint32_t)(wave * kLoads * kRowsPerLoad + kk) * (uint32_t)ld + (uint32_t)row) * 4u
                            : kOobOffset;
    }
    __device__ __forceinline__ void init_frag(int lane, int frag_row) {
        const int h = lane / S;
        frag0 = (uint32_t)((h * R + ((frag_row + lane % S) ^ turn(h))) * 4);
    }
    __device__ __forceinline__ void issue_one(uint32_t st, int k0, int wave, int i) const {
        dma16(rsrc, voff, (uint32_t)(k0 + i * kRowsPerLoad) * k_step,
              st + (uint32_t)((wave * kLoads + i) * 1024));
    }
    // element m: k = 8 ks + 64 / S m + lane / S
    __device__ __forceinline__ f32x4 frag4(const char *st, int x, int ks) const {
        const char *p = st + (frag0 ^ (uint32_t)(x << 7)) + ks * (8 * R * 4);
        f32x4 v = {};
#pragma unroll
        for (int m = 0; m < S / 8; ++m) v[m] = *(const float *)(p + m * (64 / S * R * 4));
        return v;
    }
};

enum { F32_PLAIN = 0, F32_RELU = 1, F32_MASK = 2, F32_COMBINE = 3 };   // (see gemm_rows.hip)

// MFMA tiles of S x S, S 32 or 16
__device__ __forceinline__ f32x16 mfma_f32(float p, float q, f32x16 c) {
    return __builtin_amdgcn_mfma_f32_32x32x2f32(p, q, c, 0, 0, 0);
}
__device__ __forceinline__ f32x4 mfma_f32(float p, float q, f32x4 c) {
    return __builtin_amdgcn_mfma_f32_16x16x4f32(p, q, c, 0, 0, 0);
}

// R: RouterWgradArgs, parts of the router's weight gradient in blocks behind those of a weight gradient of the experts', or
// nothing.  Two kernels, for those blocks take twice the registers (one kernel / two, us of a pass: 826 x 1824 x 1280, 128
// experts 2156 / 2075, 2088 x 496 x 5040, 128 experts 2131 / 2012).
struct NoRouterWgrad {};

template <int S, int IP, int WP, int IQ, int WQ, int STAGES, bool Q_TRANS, bool P_TRANS, int EPI, typename R>
__global__ __launch_bounds__(64 * WP * WQ, 2) void gemm_f32_mfma_kernel(GemmF32Args a, int tiles_q, int tiles_p, R router) {
    constexpr int NW = WP * WQ, PB = S * IP * WP, QB = S * IQ * WQ;
    constexpr int kPBytes = PB * 128, kStage = (PB + QB) * 128;
    constexpr int kAcc = S * S / 64;   // accumulators per lane and MFMA tile
    typedef typename std::conditional<S == 32, f32x16, f32x4>::type Acc;
    static_assert(S == 32 || IP * IQ == 1, "fragments lie 32 rows apart");
    __shared__ __attribute__((aligned(16))) char lds[STAGES * kStage];
    const int per_e = tiles_q * tiles_p;
    if constexpr (std::is_same<R, RouterWgradArgs>::value) {
        static_assert(STAGES * kStage >= kRwLds && NW == 4, "room for the router's blocks");
        const int beyond = (int)blockIdx.x - ((int)gridDim.x - router.blocks);
        if (beyond >= 0) return router_wgrad_block<float>(router, beyond, lds);
    }
    const int e = blockIdx.x / per_e, rem = blockIdx.x - e * per_e;
    const int pt = rem / tiles_q, qt = rem - pt * tiles_q;
    const int lim = a.kept[e];
    const int qlim = a.q_limited ? min(lim, a.Qdim) : a.Qdim;
    const int klim = a.k_limited ? min(lim, a.Kdim) : a.Kdim;
    const int q0 = qt * QB, p0 = pt * PB;
    if (q0 >= qlim) return;
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
    const int wp = wave % WP, wq = wave / WP;
    const uint32_t lds0 = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) char *)lds;
    const bool live = q0 + wq * S * IQ < qlim && p0 + wp * S * IP < a.Pdim;

    typename std::conditional<P_TRANS, F32Trans<PB, NW, S>, F32Direct<PB, NW, S>>::type op;
    typename std::conditional<Q_TRANS, F32Trans<QB, NW, S>, F32Direct<QB, NW, S>>::type oq;
    op.init_frag(lane, wp * S * IP);
    oq.init_frag(lane, wq * S * IQ);
    op.init(a.P + (size_t)e * a.p_batch, P_TRANS ? (int)a.p_ks : (int)a.p_rs, p0, a.Pdim, klim, lane, wave);
    oq.init(a.Q + (size_t)e * a.q_batch, Q_TRANS ? (int)a.q_ks : (int)a.q_rs, q0, qlim, klim, lane, wave);
    const int nk = (klim + 31) / 32;

    Acc acc[IP][IQ], total[IP][IQ];
#pragma unroll
    for (int i = 0; i < IP; ++i)
#pragma unroll
        for (int j = 0; j < IQ; ++j)
#pragma unroll
            for (int r = 0; r < kAcc; ++r) acc[i][j][r] = total[i][j][r] = 0.f;

    constexpr int kLoads = decltype(op)::kLoads + decltype(oq)::kLoads;
    // With two stages no step past the end is loaded: a weight gradient of few rows has one step per tile, and another one
    // took 3-6 % of the launch (96 experts of 576 x 2264, 253 tokens: 137 / 133 us).  With more stages the wait counts
    // need them; they are never read.
    auto issue = [&](int kt) {
        if (STAGES == 2 && kt >= nk) return;
        const uint32_t at = lds0 + (uint32_t)(kt % STAGES * kStage);
#pragma unroll
        for (int i = 0; i < decltype(op)::kLoads; ++i) op.issue_one(at, kt * 32, wave, i);
#pragma unroll
        for (int i = 0; i < decltype(oq)::kLoads; ++i) oq.issue_one(at + kPBytes, kt * 32, wave, i);
    };
#pragma unroll
    for (int st = 0; st < STAGES - 1; ++st) issue(st);
    for (int kt = 0; kt < nk; ++kt) {
        rows_wait_vmcnt<(STAGES - 2) * kLoads>();
        __syncthreads();   // step kt has landed, step kt - 1 is read
        issue(kt + STAGES - 1);
        if (!live) continue;
        const char *sp = lds + kt % STAGES * kStage, *sq = sp + kPBytes;
        if (kt != 0 && kt % (kF32Flush / 32) == 0) {
#pragma unroll
            for (int i = 0; i < IP; ++i)
#pragma unroll
                for (int j = 0; j < IQ; ++j)
#pragma unroll
                    for (int r = 0; r < kAcc; ++r) {
                        total[i][j][r] += acc[i][j][r];
                        acc[i][j][r] = 0.f;
                    }
        }
#pragma unroll
        for (int ks = 0; ks < 4; ++ks) {
            f32x4 fp[IP], fq[IQ];
#pragma unroll
            for (int i = 0; i < IP; ++i) fp[i] = op.frag4(sp, i, ks);
#pragma unroll
            for (int j = 0; j < IQ; ++j) fq[j] = oq.frag4(sq, j, ks);
#pragma unroll
            for (int m = 0; m < S / 8; ++m)
#pragma unroll
                for (int i = 0; i < IP; ++i)
#pragma unroll
                    for (int j = 0; j < IQ; ++j) acc[i][j] = mfma_f32(fp[i][m], fq[j][m], acc[i][j]);
        }
    }
    rows_wait_vmcnt<0>();   // the trailing loads
    if (!live) return;
    // a lane holds, for row q = lane % S of each tile, columns 256 / S g + 4 (lane / S) .. + 3
    float *Cout = a.Cout + (size_t)e * a.c_batch;
    const float *mask = EPI == F32_MASK ? a.mask + (size_t)e * a.c_batch : nullptr;
#pragma unroll
    for (int j = 0; j < IQ; ++j) {
        const int q = q0 + (wq * IQ + j) * S + lane % S;
        if (q >= qlim) continue;
        uint32_t row_idx = 0;   // index of the token's first hidden unit in the dropout stream
        if (EPI == F32_RELU && a.nz.dropout)
            row_idx = (uint32_t)a.slot_token[(size_t)e * a.slots + q] * (uint32_t)a.Pdim;
        int tok = 0;
        float gate = 0.f;
        if (EPI == F32_COMBINE) {
            tok = a.slot_token[(size_t)e * a.slots + q];
            gate = a.slot_gate[(size_t)e * a.slots + q];
        }
#pragma unroll
        for (int i = 0; i < IP; ++i)
#pragma unroll
            for (int g = 0; g < kAcc / 4; ++g) {
                const int p = p0 + (wp * IP + i) * S + 256 / S * g + lane / S * 4;
                if (p >= a.Pdim) continue;   // Pdim is a multiple of 4: four columns are in or out
                float v[4];
#pragma unroll
                for (int r = 0; r < 4; ++r) v[r] = total[i][j][4 * g + r] + acc[i][j][4 * g + r];
                const size_t at = (size_t)q * a.ldc + p;
                if (EPI == F32_RELU) {
#pragma unroll
                    for (int r = 0; r < 4; ++r) v[r] = v[r] > 0.f ? v[r] : 0.f;
                    if (a.nz.dropout) {   // Sec. 2.4: expert dropout on the hidden activation
#pragma unroll
                        for (int r = 0; r < 4; ++r)
                            v[r] = dropout_keeps(a.nz, row_idx + (uint32_t)(p + r)) ? v[r] * a.nz.drop_scale : 0.f;
                    }
                }
                if (EPI == F32_MASK) {   // a unit passes the gradient iff it was active and survived dropout
                    const float4 m = *(const float4 *)(mask + at);
                    v[0] = m.x > 0.f ? v[0] * a.nz.drop_scale : 0.f;
                    v[1] = m.y > 0.f ? v[1] * a.nz.drop_scale : 0.f;
                    v[2] = m.z > 0.f ? v[2] * a.nz.drop_scale : 0.f;
                    v[3] = m.w > 0.f ? v[3] * a.nz.drop_scale : 0.f;
                }
                *(float4 *)(Cout + at) = make_float4(v[0], v[1], v[2], v[3]);
                if (EPI == F32_COMBINE)
                    *(float4 *)(a.y + (size_t)tok * a.ldc + p) =
                        make_float4(v[0] * gate, v[1] * gate, v[2] * gate, v[3] * gate);
            }
    }
}

template <int S, int IP, int WP, int IQ, int WQ, int STAGES, bool Q_TRANS, bool P_TRANS, int EPI>
static hipError_t f32_launch(const GemmF32Args &a, int E, const RouterWgradArgs &parts, hipStream_t s) {
    const int tq = (int)ceil_div(a.Qdim, S * IQ * WQ), tp = (int)ceil_div(a.Pdim, S * IP * WP);
    auto launch = [&](auto kern, auto router) {
        hipLaunchKernelGGL(kern, dim3((unsigned)(tq * tp * E + parts.blocks)), dim3(64 * WP * WQ), 0, s, a, tq, tp, router);
        return hipGetLastError();
    };
    if constexpr (Q_TRANS)
        if (parts.blocks)
            return launch(gemm_f32_mfma_kernel<S, IP, WP, IQ, WQ, STAGES, Q_TRANS, P_TRANS, EPI, RouterWgradArgs>, parts);
    return launch(gemm_f32_mfma_kernel<S, IP, WP, IQ, WQ, STAGES, Q_TRANS, P_TRANS, EPI, NoRouterWgrad>, NoRouterWgrad{});
}

template <bool Q_TRANS, bool P_TRANS, int EPI>
static hipError_t f32_mfma(const GemmF32Args &a, int E, hipStream_t s, const RouterWgradArgs &parts = {}) {
    // 64 x 64 keeps the chip even (a 128 x 128 tile takes 573 instead of 364 us in the second GEMM of
    // 32 experts x 256 tokens x 768 x 3072); twice as wide is 2-8 % faster where there are many tiles.
    if (E * ceil_div(a.Qdim, 64) * ceil_div(a.Pdim, 128) >= 1024)
        return f32_launch<32, 2, 2, 1, 2, 2, Q_TRANS, P_TRANS, EPI>(a, E, parts, s);
    // Few tiles: a 64 x 64 tile keeps one CU's matrix cores busy for 1024 cycles per 32 k, whatever the others do.
    // Tiles of 32 x 32, a quarter of 16 x 16 per wave, spread over four times as many (us per forward + backward
    // pass, 64 x 64 / 32 x 32: 256 x 64 x 256, 4 experts 71 / 56; 1000 x 512 x 1536, 8 experts 244 / 219; 512 x 768 x
    // 3072, 4 experts 387 / 310; all products at 384 tiles or beside it, 3000 x 256 x 512, 8 experts: 132 / 135).  With
    // 385 to 700 tiles either may win: the limit at 700 instead, 2000 x 256 x 1024, 8 experts 153 -> 156, 700 x 128 x 512,
    // 32 experts 74 -> 76, 1000 x 512 x 1536 224 -> 212.
    // (Four waves that take a quarter of the k each of one 32 x 32: 2-8 % less per pass, but other sums than the
    // larger tiles'.)
    if (E * ceil_div(a.Qdim, 64) * ceil_div(a.Pdim, 64) <= 384)
        return f32_launch<16, 1, 2, 1, 2, 4, Q_TRANS, P_TRANS, EPI>(a, E, parts, s);
    return f32_launch<32, 1, 2, 1, 2, 2, Q_TRANS, P_TRANS, EPI>(a, E, parts, s);
}

// The matrix-core kernel addresses one expert's matrices through 32-bit buffer descriptors, and all of a
// product's tiles (64 x 128, 256 threads, or half of that) lie in one dimension of the grid.
bool gemm_f32_on_mfma(const Workspace &w, int64_t Qdim, int64_t Pdim) {
    const double d = (double)w.d, f1 = (double)w.f1, C = (double)w.C, most = fmax(fmax(d * f1, C * d), C * f1) * 4.;
    return most < 2147483647. && w.E * ceil_div(Qdim, 64) * ceil_div(Pdim, 128) * 256 <= kMaxGridThreads;
}

static hipError_t gemm_f32(GemmKind kind, const Workspace &w, char *ws, const void *W_in, const void *W_out,
                           void *dW_in, void *dW_out, void *y, const RouterWgradArgs &parts, hipStream_t s) {
    const long d = w.d, f = w.f, f1 = w.f1, C = w.C;
    GemmF32Args a{};
    a.kept = (const int32_t *)(ws + w.kept);
    a.slot_token = (const int32_t *)(ws + w.slot_token);
    a.slots = C;
    a.slot_gate = (const float *)(ws + w.slot_gate);
    a.y = (float *)y;
    a.nz = w.noise;
    const float *Xd = (const float *)(ws + w.Xd);
    float *A = (float *)(ws + w.A);
    float *O = (float *)(ws + w.O);
    const float *dO = (const float *)(ws + w.dO);
    float *dH = (float *)(ws + w.dH);
    float *dXd = (float *)(ws + w.dXd);
    const char *name = "";
    switch (kind) {
    case GEMM_FWD1:
        name = w.geglu ? "gemm1_fwd" : "gemm1_fwd_relu";
        a.Q = Xd; a.q_batch = C * d; a.q_rs = d; a.q_ks = 1;
        a.P = (const float *)W_in; a.p_batch = d * f1; a.p_rs = 1; a.p_ks = f1;
        a.Cout = w.geglu ? (float *)(ws + w.H) : A; a.c_batch = C * f1; a.ldc = f1;
        a.Qdim = C; a.Pdim = f1; a.Kdim = d; a.q_limited = 1; a.epi = w.geglu ? 0 : 1;
        break;
    case GEMM_FWD2:
        name = "gemm2_fwd";
        a.Q = A; a.q_batch = C * f; a.q_rs = f; a.q_ks = 1;
        a.P = (const float *)W_out; a.p_batch = f * d; a.p_rs = 1; a.p_ks = d;
        a.Cout = O; a.c_batch = C * d; a.ldc = d;
        a.Qdim = C; a.Pdim = d; a.Kdim = f; a.q_limited = 1;
        break;
    case GEMM_DGRAD2:
        name = w.geglu ? "gemm2_dgrad" : "gemm2_dgrad_relumask";
        a.Q = dO; a.q_batch = C * d; a.q_rs = d; a.q_ks = 1;
        a.P = (const float *)W_out; a.p_batch = f * d; a.p_rs = d; a.p_ks = 1;
        a.Cout = w.geglu ? (float *)(ws + w.dA) : dH; a.c_batch = C * f; a.ldc = f; a.mask = A;
        a.Qdim = C; a.Pdim = f; a.Kdim = d; a.q_limited = 1; a.epi = w.geglu ? 0 : 2;
        break;
    case GEMM_DGRAD1:
        name = "gemm1_dgrad";
        a.Q = dH; a.q_batch = C * f1; a.q_rs = f1; a.q_ks = 1;
        a.P = (const float *)W_in; a.p_batch = d * f1; a.p_rs = f1; a.p_ks = 1;
        a.Cout = dXd; a.c_batch = C * d; a.ldc = d;
        a.Qdim = C; a.Pdim = d; a.Kdim = f1; a.q_limited = 1;
        break;
    case GEMM_WGRAD2:
        name = "gemm2_wgrad";
        a.Q = A; a.q_batch = C * f; a.q_rs = 1; a.q_ks = f;
        a.P = dO; a.p_batch = C * d; a.p_rs = 1; a.p_ks = d;
        a.Cout = (float *)dW_out; a.c_batch = f * d; a.ldc = d;
        a.Qdim = f; a.Pdim = d; a.Kdim = C; a.k_limited = 1;
        break;
    case GEMM_WGRAD1:
        name = "gemm1_wgrad";
        a.Q = Xd; a.q_batch = C * d; a.q_rs = 1; a.q_ks = d;
        a.P = dH; a.p_batch = C * f1; a.p_rs = 1; a.p_ks = f1;
        a.Cout = (float *)dW_in; a.c_batch = d * f1; a.ldc = f1;
        a.Qdim = d; a.Pdim = f1; a.Kdim = C; a.k_limited = 1;
        break;
    }
    if (a.Qdim == 0) return hipSuccess;   // capacity 0 and a slot-indexed output: nothing to do
    ProfScope ps(name, s);
    if (gemm_f32_on_mfma(w, a.Qdim, a.Pdim)) {
        const int E = (int)w.E;
        switch (kind) {
        case GEMM_FWD1:
            return w.geglu ? f32_mfma<false, true, F32_PLAIN>(a, E, s) : f32_mfma<false, true, F32_RELU>(a, E, s);
        case GEMM_FWD2:
            return w.combine_in_gemm ? f32_mfma<false, true, F32_COMBINE>(a, E, s) : f32_mfma<false, true, F32_PLAIN>(a, E, s);
        case GEMM_DGRAD2:
            return w.geglu ? f32_mfma<false, false, F32_PLAIN>(a, E, s) : f32_mfma<false, false, F32_MASK>(a, E, s);
        case GEMM_DGRAD1: return f32_mfma<false, false, F32_PLAIN>(a, E, s);
        case GEMM_WGRAD2:
        case GEMM_WGRAD1: return f32_mfma<true, true, F32_PLAIN>(a, E, s, parts);
        }
    }
    dim3 grid((unsigned)ceil_div(a.Pdim, kF32Tile), (unsigned)ceil_div(a.Qdim, kF32Tile),
              (unsigned)w.E);
    hipLaunchKernelGGL(gemm_f32_kernel, grid, dim3(256), 0, s, a);
    return hipGetLastError();
}

hipError_t launch_gemm_f32(GemmKind kind, const Workspace &w, char *ws, const void *W_in,
                           const void *W_out, void *dW_in, void *dW_out, const TokenMajor &tm,
                           hipStream_t s) {
    return gemm_f32(kind, w, ws, W_in, W_out, dW_in, dW_out, tm.y, RouterWgradArgs{}, s);
}

hipError_t launch_gemm_f32_wgrad1(const Workspace &w, char *ws, void *dW_in, const RouterWgradArgs &parts, hipStream_t s) {
    return gemm_f32(GEMM_WGRAD1, w, ws, nullptr, nullptr, dW_in, nullptr, nullptr, parts, s);
}

}  // namespace sw
