// Weight gradients of the experts (bf16 MFMA, fp32 accumulation), persistent blocks:
//     dW_e[q][p] = sum over the expert's kept slots k of Q_e[k][q] P_e[k][p].
//
// What bounds it: a tile has few k steps (an expert's slots: 4 .. 10 steps of 64) and then 196 KB to
// store, and its registers and LDS leave no room for a second block on the CU, so with a block per
// tile neither the start (launch, first loads) nor the store has anything beside it.  Here a block
// walks over the tiles of its XCD's experts: the last step of a tile loads the first step of the next one,
// which lands during the epilogue, and the stores retire behind the next tile's products.
//
// Eight waves, 256 x 384 or 384 x 256 accumulators, 64 k per step in two LDS stages of 80 KB filled
// by direct loads.  The epilogue turns a wave's rows around in the stage that the tile's last step has
// read; the other stage holds the next tile's first step by then.
//
// us per launch, first / second gradient, a block per tile -> here: 128 experts of 768 x 3072, 512 slots
// 344 / 340 -> 299 / 310, 64 slots 151 / 152 -> 119 / 125, two experts with tokens 123 / 151 -> 102 / 119; 64 experts
// of 4096 x 10240, 256 slots 2340 / 2170 -> 1990 / 1980.  A step of 64 k takes 4500 .. 5800 cycles for 3072 of
// MFMA: both operands are read transposed (8 bytes per lane), 1800 cycles of LDS reads and 640 of writes by the
// loads; the clock is 1.8 .. 2.0 GHz under the products' power.  (256 x 256 here: 348 / 350.)
#include "common.h"
#include "lds_operands.h"
#include "rows_operands.h"

namespace sw {

struct WgradArgs {
    const bf16 *Q, *P;          // per expert q_batch / p_batch elements: [slot][ldq], [slot][ldp]
    bf16 *Cout;                 // [E][ldq][ldp]
    size_t q_batch, p_batch;
    int ldq, ldp;               // = rows and columns of a gradient
    const int32_t *kept;
    int tiles_q, tiles_p, E;
    int by_expert;              // every eighth expert is an XCD's, else an eighth of the tiles
};

template <int IP, int WP, int IQ, int WQ>
__global__ __launch_bounds__(512, 2) void gemm_wgrad_kernel(WgradArgs a) {
    constexpr int NW = WP * WQ, BK = 64, PB = 32 * IP * WP, QB = 32 * IQ * WQ;
    constexpr int kPBytes = PB * BK * 2, kStage = (PB + QB) * BK * 2;
    static_assert(NW == 8 && 2 * kStage <= 160 * 1024, "two stages");
    extern __shared__ __attribute__((aligned(16))) char lds[];
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
    const int wp = wave % WP, wq = wave / WP;
    const uint32_t lds0 = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) char *)lds;
    // block b runs on XCD b mod 8 and takes every (blocks per XCD)-th of its tiles
    const int per_e = a.tiles_p * a.tiles_q, total = per_e * a.E, xcd = (int)blockIdx.x & 7;
    const int per = (total + 7) >> 3, stride = (int)gridDim.x >> 3;
    const int lo = a.by_expert ? 0 : xcd * per, end = a.by_expert ? (a.E - xcd + 7) / 8 * per_e : min(lo + per, total);
    int n = lo + ((int)blockIdx.x >> 3);
    if (n >= end) return;

    auto locate = [&](int at, int &e, int &q0, int &p0) {
        e = at / per_e;
        const int rem = at - e * per_e;
        if (a.by_expert) e = e * 8 + xcd;
        int pt, qt;   // the dimension with fewer tiles runs fastest: sharers of the larger operand are neighbours
        if (a.tiles_q <= a.tiles_p) {
            pt = rem / a.tiles_q;
            qt = rem - pt * a.tiles_q;
        } else {
            qt = rem / a.tiles_p;
            pt = rem - qt * a.tiles_p;
        }
        q0 = qt * QB;
        p0 = pt * PB;
    };
    RowsTrans<PB, NW> op;
    RowsTrans<QB, NW> oq;
    constexpr int kLoads = decltype(op)::kLoads + decltype(oq)::kLoads;
    op.init_frag(lane, wp * 32 * IP);
    oq.init_frag(lane, wq * 32 * IQ);
    // operands of tile `at` (past the last one, and without slots: empty descriptors); returns its k steps
    auto point = [&](int at) {
        int e = 0, q0 = 0, p0 = 0, klim = 0;
        if (at < end) {
            locate(at, e, q0, p0);
            // (a scalar load: a vector load's wait would also wait for the loads and stores in flight)
            klim = *((const __attribute__((address_space(4))) int32_t *)(uintptr_t)a.kept + e);
        }
        op.init(a.P + (size_t)e * a.p_batch, a.ldp, p0, a.ldp, klim, lane, wave);
        oq.init(a.Q + (size_t)e * a.q_batch, a.ldq, q0, a.ldq, klim, lane, wave);
        return (klim + BK - 1) / BK;
    };
    auto issue_load = [&](uint32_t at, int kt, int i) {
        if (i < decltype(op)::kLoads) op.issue_one(at, kt * BK, wave, i);
        else oq.issue_one(at + kPBytes, kt * BK, wave, i - decltype(op)::kLoads);
    };

    // one k step from stage st; the other stage is filled with step `kt` of the tile the operands point at
    auto step = [&](auto first, f32x16 (&acc)[IP][IQ], int st, int kt) {
        const char *sp = lds + st * kStage, *sq = sp + kPBytes;
        const uint32_t fill = lds0 + (uint32_t)((st ^ 1) * kStage);
#pragma unroll
        for (int ks = 0; ks < BK / 16; ++ks) {
            bf16x8 fp[IP], fq[IQ];
#pragma unroll
            for (int i = 0; i < IP; ++i) fp[i] = op.frag(sp, i, ks);
#pragma unroll
            for (int j = 0; j < IQ; ++j) fq[j] = oq.frag(sq, j, ks);
#pragma unroll
            for (int i = 0; i < kLoads; ++i)   // over three of the four sub-steps
                if (i * 3 / kLoads == ks) issue_load(fill, kt, i);
#pragma unroll
            for (int i = 0; i < IP; ++i)
#pragma unroll
                for (int j = 0; j < IQ; ++j) {
                    if (decltype(first)::value && ks == 0) {
                        const f32x16 zero = {};
                        acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fp[i], fq[j], zero, 0, 0, 0);
                    } else {
                        acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fp[i], fq[j], acc[i][j], 0, 0, 0);
                    }
                }
        }
    };

    // an odd number of chunks per row, as in rows_operands.h; the 8-byte writes of rows 8 apart meet in a bank here too
    // (0.20 of the LDS cycles at 512 slots of 768 x 3072, 0.27 at 256 of 4096 x 10240)
    constexpr int kPitch = 64 * IP + 16, kChunks = 4 * IP, kPasses = 2 * IP, kStores = IQ * kPasses;
    static_assert(kStores <= 63 && NW * 32 * kPitch <= kStage, "the turn-around buffers fit a stage");
    int nk = point(n), st = 0;
#pragma unroll
    for (int i = 0; i < kLoads; ++i) issue_load(lds0, 0, i);
    bool stores = false;   // the tile before has stores in flight, younger than this tile's first loads
    while (n < end) {
        int e, q0, p0;
        locate(n, e, q0, p0);
        int next_nk = 0;
        // The stores' lane id goes through an empty asm: addresses made from it would be kept in registers over
        // the k loop, which has none to spare.
        int lane_e = lane;
        asm volatile("" : "+v"(lane_e));
        const auto crsrc = __builtin_amdgcn_make_buffer_rsrc(a.Cout + (size_t)e * a.ldq * a.ldp, 0,
                                                             (int)((uint32_t)a.ldq * (uint32_t)a.ldp * 2u), 0x00020000);
        if (nk == 0) {   // an expert without tokens: zeros, whole rows of the tile at a time
            __syncthreads();   // the stage to fill is read (the epilogue before may have used it)
            next_nk = point(n + stride);
#pragma unroll
            for (int i = 0; i < kLoads; ++i) issue_load(lds0 + (uint32_t)((st ^ 1) * kStage), 0, i);
            st ^= 1;
#pragma unroll
            for (int x = 0; x < kStores; ++x) {
                const int at = (wave * kStores + x) * 64 + lane_e, row = q0 + at / (PB / 8), p = p0 + at % (PB / 8) * 8;
                const bool in = row < a.ldq && p < a.ldp;
                const uint32_t off = in ? ((uint32_t)row * (uint32_t)a.ldp + (uint32_t)p) * 2u : kOobOffset;
                __builtin_amdgcn_raw_buffer_store_b128(u32x4{0u, 0u, 0u, 0u}, crsrc, (int)off, 0, 0);
            }
            stores = true;
            n += stride;
            nk = next_nk;
            continue;
        }
        f32x16 acc[IP][IQ];
        auto advance = [&](auto first, int kt) {
            if (decltype(first)::value && stores) rows_wait_vmcnt<kStores>();
            else rows_wait_vmcnt<0>();
            __syncthreads();   // the step has landed for all waves; the other stage is read
            int load = kt + 1;
            if (load == nk) {
                next_nk = point(n + stride);
                load = 0;
            }
            step(first, acc, st, load);
            st ^= 1;
        };
        advance(std::true_type{}, 0);
        for (int kt = 1; kt < nk; ++kt) advance(std::false_type{}, kt);
        __syncthreads();   // all waves have read the last stage (st ^ 1)

        // Epilogue: 32 rows at a time through LDS of the wave's own, see gemm_rows.hip
        char *ep = lds + (st ^ 1) * kStage + wave * 32 * kPitch;
        const int pw = p0 + wp * 32 * IP, wrow = lane_e & 31;
        const uint32_t c_step = 64u * (uint32_t)a.ldp;   // bytes of 32 rows
        uint32_t cvoff[kPasses];   // of the lane's piece in pass x, first 32 rows of the wave,
        int left[kPasses];         // and the rows from there to the last one (offsets of rows past it may wrap)
#pragma unroll
        for (int x = 0; x < kPasses; ++x) {
            const int at = x * 64 + lane_e, row = at / kChunks, p = pw + (at - row * kChunks) * 8;
            cvoff[x] = ((uint32_t)(q0 + wq * IQ * 32 + row) * (uint32_t)a.ldp + (uint32_t)p) * 2u;
            left[x] = p < a.ldp ? a.ldq - (q0 + wq * IQ * 32 + row) : 0;
        }
#pragma unroll
        for (int j = 0; j < IQ; ++j) {
#pragma unroll
            for (int i = 0; i < IP; ++i)
#pragma unroll
                for (int g = 0; g < 4; ++g) {
                    const uint2 o = make_uint2(pack_bf16(acc[i][j][4 * g], acc[i][j][4 * g + 1]),
                                               pack_bf16(acc[i][j][4 * g + 2], acc[i][j][4 * g + 3]));
                    *(uint2 *)(ep + wrow * kPitch + ((i * 4 + g) << 4) + ((lane_e >> 5) << 3)) = o;
                }
#pragma unroll
            for (int x = 0; x < kPasses; ++x) {
                const int at = x * 64 + lane_e, row = at / kChunks, c = at - row * kChunks;
                const u32x4 val = *(const u32x4 *)(ep + row * kPitch + (c << 4));
                const uint32_t off = 32 * j < left[x] ? cvoff[x] + (uint32_t)j * c_step : kOobOffset;
                __builtin_amdgcn_raw_buffer_store_b128(val, crsrc, (int)off, 0, 0);
            }
        }
        stores = true;
        n += stride;
        nk = next_nk;
    }
    rows_wait_vmcnt<0>();   // the loads past the last tile (zeros)
}

template <int IP, int WP, int IQ, int WQ> static hipError_t wgrad_launch(WgradArgs a, int E, hipStream_t s) {
    auto kern = gemm_wgrad_kernel<IP, WP, IQ, WQ>;
    constexpr int PB = 32 * IP * WP, QB = 32 * IQ * WQ, lds = 2 * (PB + QB) * 128;
    static PerDeviceOnce once;
    static int cu_count[kMaxDevices];
    int dev = -1;
    if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= kMaxDevices) return hipErrorInvalidDevice;
    hipError_t err = once_per_device(once, [&] {
        int cus = 0;
        hipError_t e = hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev);
        cu_count[dev] = cus >= 8 ? cus / 8 * 8 : 8;
        if (e != hipSuccess) return e;
        return hipFuncSetAttribute((const void *)kern, hipFuncAttributeMaxDynamicSharedMemorySize, lds);
    });
    if (err != hipSuccess) return err;
    a.tiles_q = (int)ceil_div(a.ldq, QB);
    a.tiles_p = (int)ceil_div(a.ldp, PB);
    a.E = E;
    // an expert's tiles on one XCD, whose L2 then holds its operands; neighbours, which a skewed router likes
    // alike, on different ones
    a.by_expert = E % 8 == 0 || E >= 64;
    const int64_t per_e = (int64_t)a.tiles_q * a.tiles_p;
    const int64_t blocks = a.by_expert ? ceil_div(E, 8) * per_e * 8 : ceil_div(per_e * E, 8) * 8;
    hipLaunchKernelGGL(kern, dim3((unsigned)(blocks < cu_count[dev] ? blocks : cu_count[dev])), dim3(512), lds, s, a);
    return hipGetLastError();
}

hipError_t launch_gemm_wgrad(GemmKind kind, const Workspace &w, char *ws, void *dW_in, void *dW_out, int tile,
                             hipStream_t s) {
    const bool two = kind == GEMM_WGRAD2;
    ProfScope ps(two ? "gemm2_wgrad" : "gemm1_wgrad", s);
    WgradArgs a{};
    a.kept = (const int32_t *)(ws + w.kept);
    a.Q = (const bf16 *)(ws + (two ? w.A : w.Xd)); a.ldq = (int)(two ? w.f : w.d); a.q_batch = (size_t)w.C * a.ldq;
    a.P = (const bf16 *)(ws + (two ? w.dO : w.dH)); a.ldp = (int)(two ? w.d : w.f1); a.p_batch = (size_t)w.C * a.ldp;
    a.Cout = (bf16 *)(two ? dW_out : dW_in);
    if (tile == ROWS_384x256) return wgrad_launch<4, 2, 3, 4>(a, (int)w.E, s);
    return wgrad_launch<3, 4, 4, 2>(a, (int)w.E, s);
}

}  // namespace sw
