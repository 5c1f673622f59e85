// Gradient of the router's weights on the bf16 matrix cores (bf16 tokens, a multiple of 4 experts):
//     part[split][k][e] = sum over the split's tokens t of x[t][k] (hi[t][e] + lo[t][e]),
// hi + lo the two bf16 terms of the logits' gradient that router_bwd.hip or router_dlogits_kernel leaves; with input
// jitter x is replaced by the hi and mid planes of x * m that the forward pass leaves.  All terms go into one fp32
// sum; reduce_dWr_split_kernel adds up the splits in order.
//
// What bounds it: x and the terms once from HBM, and the parts, written and read again.  A block takes 256 k x 128
// experts of one range of tokens, eight waves of 64 x 64, 32 tokens per step through LDS stages filled by direct loads;
// blocks of one range run on one XCD, whose L2 then holds its terms.  As many ranges as give every CU a block.
// us, the persistent 256 x 256 kernel with hi and lo in columns of their own / here, parts and their sums (with the events'
// 4 each): 65536 x 768, 128 experts 50 + 14 / 43 + 10, with jitter 87 + 26 / 75 + 10; 8192 26 + 11 / 17 + 8; 16384 x
// 4096, 64 experts 96 + 26 / 47 + 7.
#include "common.h"
#include "lds_operands.h"
#include "rows_operands.h"

namespace sw {

struct RouterDwrArgs {
    const bf16 *x, *dl;      // [T][ldx], [etiles][T][256]
    float *part;             // [etiles][nsplit][d][128]
    int ldx, plane;          // elements of a row, and from one plane of it to the next
    int T, d, E, tps, nsplit, tiles_q, per_tile;   // per_tile: blocks of a tile of 128 experts
};

template <int PLANES> __global__ __launch_bounds__(512, 2) void router_dWr_mfma_kernel(RouterDwrArgs a) {
    constexpr int NW = 8, BK = 32, STAGES = PLANES == 1 ? 4 : 3, kOp = 256 * BK * 2, kStage = (PLANES + 1) * kOp;
    __shared__ __attribute__((aligned(16))) char lds[STAGES * kStage];
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
    const int wp = wave & 1, wq = wave >> 1;
    const uint32_t lds0 = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) char *)lds;
    // block b runs on XCD b mod 8
    const int et = blockIdx.y, per = a.per_tile >> 3, at = ((int)blockIdx.x & 7) * per + ((int)blockIdx.x >> 3);
    const int split = at / a.tiles_q, q0 = (at - split * a.tiles_q) * 256;
    if (split >= a.nsplit) return;
    const int t0 = split * a.tps, klim = min(a.tps, a.T - t0), nk = (klim + BK - 1) / BK;
    const bool live = et * 128 + wp * 64 < a.E && q0 + wq * 64 < a.d;

    typedef RowsTrans<256, NW, BK> Operand;
    Operand ox[PLANES], ol;
    constexpr int kLoads = (PLANES + 1) * Operand::kLoads;
#pragma unroll
    for (int s = 0; s < PLANES; ++s) {
        ox[s].init(a.x + (size_t)t0 * a.ldx + s * a.plane, a.ldx, q0, a.d, klim, lane, wave);
        ox[s].init_frag16(lane, wq * 64);
    }
    ol.init(a.dl + ((size_t)et * a.T + t0) * 256, 256, 0, 256, klim, lane, wave);
    ol.init_frag16(lane, wp * 64);
    auto issue = [&](int kt) {   // (steps past the end: never read)
        const uint32_t st = lds0 + (uint32_t)(kt % STAGES * kStage);
#pragma unroll
        for (int s = 0; s < PLANES; ++s)
#pragma unroll
            for (int i = 0; i < Operand::kLoads; ++i) ox[s].issue_one(st + (uint32_t)(s * kOp), kt * BK, wave, i);
#pragma unroll
        for (int i = 0; i < Operand::kLoads; ++i) ol.issue_one(st + (uint32_t)(PLANES * kOp), kt * BK, wave, i);
    };
    f32x4 acc[4][4];
#pragma unroll
    for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int j = 0; j < 4; ++j) acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int s = 0; s < STAGES - 1; ++s) issue(s);
    for (int kt = 0; kt < nk; ++kt) {
        rows_wait_vmcnt<(STAGES - 2) * kLoads>();
        __syncthreads();   // step kt has landed, step kt - 1 is read
        issue(kt + STAGES - 1);
        if (!live) continue;
        const char *st = lds + kt % STAGES * kStage;
        bf16x8 fl[8];   // hi, then lo
#pragma unroll
        for (int i = 0; i < 8; ++i) fl[i] = ol.frag16(st + PLANES * kOp, i < 4 ? i : 4 + i, 0);
#pragma unroll
        for (int j = 0; j < 4; ++j)
#pragma unroll
            for (int s = 0; s < PLANES; ++s) {
                const bf16x8 fx = ox[s].frag16(st + s * kOp, j, 0);
#pragma unroll
                for (int i = 0; i < 8; ++i)
                    acc[i & 3][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(fl[i], fx, acc[i & 3][j], 0, 0, 0);
            }
    }
    rows_wait_vmcnt<0>();   // the trailing loads
    if (!live) return;
    // a lane holds, of k lane % 16 of each tile, experts 4 (lane / 16) .. + 3
    float *out = a.part + ((size_t)et * a.nsplit + split) * a.d * 128 + wp * 64 + (lane >> 4) * 4;
#pragma unroll
    for (int j = 0; j < 4; ++j) {
        const int k = q0 + wq * 64 + j * 16 + (lane & 15);
        if (k < a.d)
#pragma unroll
            for (int i = 0; i < 4; ++i) *(f32x4 *)(out + (size_t)k * 128 + i * 16) = acc[i][j];
    }
}

// Tokens per range: every CU a block, at least 64 tokens, at most 128 ranges (the sums read them all).
int64_t router_dwr_tokens(const Workspace &w) {
    int64_t splits = 256 / (ceil_div(w.d, 256) * w.etiles);
    splits = splits < 1 ? 1 : splits > 128 ? 128 : splits;
    const int64_t t = ceil_div(ceil_div(w.T, splits), 32) * 32;
    return t < 64 ? 64 : t;
}

hipError_t launch_router_dWr_mfma(const Workspace &w, const void *x, char *ws, hipStream_t s) {
    ProfScope ps("router_dWr_mfma", s);
    const bool jitter = w.noise.jitter;
    RouterDwrArgs a{};
    a.x = jitter ? (const bf16 *)(ws + w.xj) : (const bf16 *)x;
    a.ldx = jitter ? (int)w.dpad_r : (int)w.d;
    a.plane = (int)w.dpad;
    a.dl = (const bf16 *)(ws + w.dl_split);
    a.part = (float *)(ws + w.dWr_part_m);
    a.T = (int)w.T; a.d = (int)w.d; a.E = (int)w.E;
    a.tps = (int)w.tps_m; a.nsplit = (int)w.nsplit_m;
    a.tiles_q = (int)ceil_div(w.d, 256);
    a.per_tile = (int)(ceil_div((int64_t)a.tiles_q * a.nsplit, 8) * 8);
    const dim3 grid((unsigned)a.per_tile, (unsigned)w.etiles);
    if (jitter) hipLaunchKernelGGL(router_dWr_mfma_kernel<2>, grid, dim3(512), 0, s, a);
    else hipLaunchKernelGGL(router_dWr_mfma_kernel<1>, grid, dim3(512), 0, s, a);
    return hipGetLastError();
}

}  // namespace sw
