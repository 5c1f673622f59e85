// Weight gradients of the experts (bf16 MFMA, fp32 accumulation), persistent blocks:
//     dW_e[q][p] = sum over the expert's kept slots k of Q_e[k][q] P_e[k][p].
//
// What bounds it: a tile has few k steps (an expert's slots: 8 .. 20 steps of 32) and then 196 KB to
// store, and its registers and LDS leave no room for a second block on the CU, so with a block per
// tile neither the start (launch, first loads) nor the store has anything beside it.  Here a block
// walks over the tiles of its XCD's experts: the loads run two steps ahead of the products, over the ends of tiles,
// and the stores retire behind the next tile's first two steps.
//
// Eight waves, 256 x 384 or 384 x 256 accumulators in MFMA tiles of 16 x 16 x 32 (see gemm_rows.hip), 32 k per step in
// three LDS stages of 40 KB filled by direct loads, and a turn-around buffer of each wave's own for the epilogue.  (Stores
// from registers, 64-byte segments of 16 rows each by lane swaps, need no buffer and leave room for a fourth stage,
// but take 330 us at Switch-Base; four waves with 192 x 256, two blocks per CU, 310 us and more load requests.)
//
// us per launch, first / second gradient, a block per tile -> 64 k in two stages, MFMA 32 x 32 x 16 -> here: 128 experts
// of 768 x 3072, 512 slots 344 / 340 -> 293 / 308 -> 291 / 300, 64 slots 151 / 152 -> 120 / 130 -> 119 / 134, two experts
// with tokens 123 / 151 -> 100 / 118 -> 100 / 118; 4096 wide (gated GELU) 424 / 213 -> 396 / 206; 64 experts of 4096 x 10240,
// 256 slots 2340 / 2170 -> 2038 / 2007 -> 2065 / 1942.  The products alone take 170 of the 290 us, with the fragment
// reads and barriers 205, with the epilogue 225; loads and stores account for the rest (with every store in one 16 KB
// window 265).
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

template <int IP, int WP, int IQ, int WQ> struct WgradShape {
    static constexpr int NW = WP * WQ, BK = 32, STAGES = 3, PB = 32 * IP * WP, QB = 32 * IQ * WQ;
    static constexpr int kPBytes = PB * BK * 2, kStage = (PB + QB) * BK * 2;
    static constexpr int kPitch = 64 * IP + 16;         // an odd number of chunks per row: no bank conflicts
    static constexpr int kTurn = 16 * kPitch;           // bytes of a wave's turn-around buffer
    static constexpr int kLds = STAGES * kStage + NW * kTurn;
    static_assert(NW == 8 && kLds <= 160 * 1024, "one block of eight waves per CU");
};

template <int IP, int WP, int IQ, int WQ>
__global__ __launch_bounds__(512, 2) void gemm_wgrad_kernel(WgradArgs a) {
    typedef WgradShape<IP, WP, IQ, WQ> S;
    constexpr int NW = S::NW, BK = S::BK, PB = S::PB, QB = S::QB;
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
    // (a scalar load: a vector load's wait would also wait for the loads and stores in flight)
    auto slots_of = [&](int e) { return *((const __attribute__((address_space(4))) int32_t *)(uintptr_t)a.kept + e); };
    RowsTrans<PB, NW, BK> op;
    RowsTrans<QB, NW, BK> oq;
    constexpr int kLoadsP = decltype(op)::kLoads, kLoads = kLoadsP + decltype(oq)::kLoads;
    op.init_frag16(lane, wp * 32 * IP);
    oq.init_frag16(lane, wq * 32 * IQ);
    // The loads run two steps ahead of the products, over the block's tiles that have slots: step load_k of tile load_n
    // (past the last one: empty descriptors, which read zeros).
    int load_n = n - stride, load_k = 0, load_nk = 0, load_st = 0;
    auto next_step = [&] {
        if (++load_k < load_nk) return;
        load_k = 0;
        int e = 0, q0 = 0, p0 = 0, klim = 0;
        while (load_n + stride < end && klim == 0) {
            load_n += stride;
            locate(load_n, e, q0, p0);
            klim = slots_of(e);
        }
        if (klim == 0) e = 0;
        load_nk = klim ? (klim + BK - 1) / BK : 0x7fffffff;
        int lane_i = lane;
        asm volatile("" : "+v"(lane_i));   // (what depends on it would stay in registers over the k loop)
        op.init(a.P + (size_t)e * a.p_batch, a.ldp, p0, a.ldp, klim, lane_i, wave);
        oq.init(a.Q + (size_t)e * a.q_batch, a.ldq, q0, a.ldq, klim, lane_i, wave);
    };
    auto issue_load = [&](int i) {
        const uint32_t at = lds0 + (uint32_t)(load_st * S::kStage);
        if (i < kLoadsP) op.issue_one(at, load_k * BK, wave, i);
        else oq.issue_one(at + S::kPBytes, load_k * BK, wave, i - kLoadsP);
    };
    auto stage_after = [](int st) { return st == S::STAGES - 1 ? 0 : st + 1; };
#pragma unroll
    for (int s = 0; s < 2; ++s) {
        next_step();
#pragma unroll
        for (int i = 0; i < kLoads; ++i) issue_load(i);
        load_st = stage_after(load_st);
    }

    // The fragments of the shorter side are held for a step, those of the other pass by, one ahead (registers).
    constexpr int kHeld = 2 * (IP < IQ ? IP : IQ), kPass = 2 * (IP < IQ ? IQ : IP);
    auto frag_held = [&](const char *st, int i) { return IP < IQ ? op.frag16(st, i, 0) : oq.frag16(st + S::kPBytes, i, 0); };
    auto frag_pass = [&](const char *st, int j) { return IP < IQ ? oq.frag16(st + S::kPBytes, j, 0) : op.frag16(st, j, 0); };
    f32x4 acc[2 * IP][2 * IQ];
    rows_wait_vmcnt<kLoads>();
    __syncthreads();
    bf16x8 held[kHeld], next = frag_pass(lds, 0);
#pragma unroll
    for (int i = 0; i < kHeld; ++i) held[i] = frag_held(lds, i);

    constexpr int kChunks = 4 * IP, kRounds = 2 * IQ, kStores = kRounds * IP;   // 16 rows and IP stores a round
    static_assert(kLoads + kStores <= 63, "the counter of loads and stores in flight");
    static_assert(kStores * NW * kWave * 8 == PB * QB, "a share of zeros is no more than a tile");
    char *ep = lds + S::STAGES * S::kStage + wave * S::kTurn;
    int st = 0;
    bool stores = false;   // the tile before has stores in flight, younger than the loads of this tile's first two steps
    for (; n < end; n += stride) {
        int e, q0, p0;
        locate(n, e, q0, p0);
        const int klim = slots_of(e), nk = (klim + BK - 1) / BK;
        // The stores' lane id goes through an empty asm: addresses made from it would be kept in registers over
        // the k loop, which has none to spare.
        int lane_e = lane;
        asm volatile("" : "+v"(lane_e));
        const auto crsrc = __builtin_amdgcn_make_buffer_rsrc(a.Cout + (size_t)e * a.ldq * a.ldp, 0,
                                                             (int)((uint32_t)a.ldq * (uint32_t)a.ldp * 2u), 0x00020000);
        if (nk == 0) {   // an expert without tokens: zeros, its gradient dealt over the tiles as plain memory
            const uint32_t chunks = (uint32_t)a.ldq * (uint32_t)a.ldp / 8u;
            const uint32_t share = ((chunks + (uint32_t)per_e - 1u) / (uint32_t)per_e + 7u) & ~7u;   // whole lines
            const uint32_t first = (uint32_t)(n % per_e) * share, last = min(first + share, chunks);
#pragma unroll
            for (int x = 0; x < kStores; ++x) {
                const uint32_t at = first + (uint32_t)((x * NW + wave) * kWave + lane_e);
                __builtin_amdgcn_raw_buffer_store_b128(u32x4{0u, 0u, 0u, 0u}, crsrc, (int)(at < last ? at * 16u : kOobOffset),
                                                       0, 0);
            }
            stores = true;
            continue;
        }
#pragma unroll
        for (int i = 0; i < 2 * IP; ++i)
#pragma unroll
            for (int j = 0; j < 2 * IQ; ++j) acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma nounroll
        for (int kt = 0; kt < nk; ++kt) {   // (one copy of the step: a first one of its own spills)
            const int st1 = stage_after(st);
            const char *cur = lds + st * S::kStage, *nxt = lds + st1 * S::kStage;
            next_step();
            op.reload_frag();
            oq.reload_frag();
#pragma unroll
            for (int j = 0; j < kPass; ++j) {
                const bool last = j == kPass - 1;
                const bf16x8 f = next;
                if (j < kLoads) issue_load(j);
                if (last) {   // the next step has landed
                    if (kt == 0 && stores) rows_wait_vmcnt<kLoads + kStores>();
                    else rows_wait_vmcnt<kLoads>();
                    __syncthreads();   // ... for all waves, and this one is read
                }
                next = last ? frag_pass(nxt, 0) : frag_pass(cur, j + 1);
                __builtin_amdgcn_sched_barrier(0);
#pragma unroll
                for (int i = 0; i < kHeld; ++i) {
                    f32x4 &c = IP < IQ ? acc[i][j] : acc[j][i];
                    c = __builtin_amdgcn_mfma_f32_16x16x32_bf16(IP < IQ ? held[i] : f, IP < IQ ? f : held[i], c, 0, 0, 0);
                }
                if (last)
#pragma unroll
                    for (int i = 0; i < kHeld; ++i) held[i] = frag_held(nxt, i);
                __builtin_amdgcn_sched_barrier(0);
            }
            load_st = stage_after(load_st);
            st = st1;
        }

        // Epilogue: 16 rows at a time through LDS of the wave's own, see gemm_rows.hip
        const int pw = p0 + wp * 32 * IP;
        const uint32_t c_step = 2u * (uint32_t)a.ldp;   // bytes of a row
        // of the lane's piece in pass x, first 16 rows of the wave (IP == 4: passes are four rows apart),
        constexpr int kPieces = IP == 4 ? 1 : IP;
        uint32_t cvoff[kPieces];
        int left[kPieces];   // and the rows from there to the last one (offsets of rows past it may wrap)
#pragma unroll
        for (int x = 0; x < kPieces; ++x) {
            const int at = x * 64 + lane_e, row = at / kChunks, p = pw + (at - row * kChunks) * 8;
            cvoff[x] = ((uint32_t)(q0 + wq * IQ * 32 + row) * (uint32_t)a.ldp + (uint32_t)p) * 2u;
            left[x] = p < a.ldp ? a.ldq - (q0 + wq * IQ * 32 + row) : 0;
        }
#pragma unroll
        for (int j = 0; j < kRounds; ++j) {
#pragma unroll
            for (int i = 0; i < 2 * IP; ++i) {
                const f32x4 v = acc[i][j];
                *(uint2 *)(ep + (lane_e & 15) * S::kPitch + (i << 5) + ((lane_e >> 4) << 3)) =
                    make_uint2(pack_bf16(v[0], v[1]), pack_bf16(v[2], v[3]));
            }
#pragma unroll
            for (int x = 0; x < IP; ++x) {
                const int y = x % kPieces, more = IP == 4 ? 4 * x : 0;   // rows
                const int at = y * 64 + lane_e, row = at / kChunks, c = at - row * kChunks;
                const u32x4 val = *(const u32x4 *)(ep + (row + more) * S::kPitch + (c << 4));
                const int rows = 16 * j + more;
                const uint32_t off = rows < left[y] ? cvoff[y] + (uint32_t)rows * c_step : kOobOffset;
                __builtin_amdgcn_raw_buffer_store_b128(val, crsrc, (int)off, 0, 0);
            }
        }
        stores = true;
    }
    rows_wait_vmcnt<0>();   // the loads past the last tile (zeros)
}

template <int IP, int WP, int IQ, int WQ> static hipError_t wgrad_launch(WgradArgs a, int E, hipStream_t s) {
    auto kern = gemm_wgrad_kernel<IP, WP, IQ, WQ>;
    typedef WgradShape<IP, WP, IQ, WQ> S;
    static PerDeviceOnce once;
    static int cu_count[kMaxDevices];
    int dev = -1;
    if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= kMaxDevices) return hipErrorInvalidDevice;
    hipError_t err = once_per_device(once, [&] {
        int cus = 0;
        hipError_t e = hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev);
        cu_count[dev] = cus >= 8 ? cus / 8 * 8 : 8;
        if (e != hipSuccess) return e;
        return hipFuncSetAttribute((const void *)kern, hipFuncAttributeMaxDynamicSharedMemorySize, S::kLds);
    });
    if (err != hipSuccess) return err;
    a.tiles_q = (int)ceil_div(a.ldq, S::QB);
    a.tiles_p = (int)ceil_div(a.ldp, S::PB);
    a.E = E;
    // an expert's tiles on one XCD, whose L2 then holds its operands; neighbours, which a skewed router likes
    // alike, on different ones
    a.by_expert = E % 8 == 0 || E >= 64;
    const int64_t per_e = (int64_t)a.tiles_q * a.tiles_p;
    const int64_t blocks = a.by_expert ? ceil_div(E, 8) * per_e * 8 : ceil_div(per_e * E, 8) * 8;
    hipLaunchKernelGGL(kern, dim3((unsigned)(blocks < cu_count[dev] ? blocks : cu_count[dev])), dim3(512), S::kLds, s, a);
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
