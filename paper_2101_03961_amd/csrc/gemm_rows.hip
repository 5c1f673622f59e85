// Grouped expert GEMMs with one tile per block (bf16 MFMA, fp32 accumulation): the products whose rows are tokens,
// and the weight gradients of layers with few or small tiles (the others: gemm_wgrad.hip, gemm_bf16.hip).
//
// The same products as gemm_bf16.hip's,
//     C_e[q][p] = sum_k Q_e(q, k) P_e(p, k),
// with tile shapes for every number of rows an expert may hold, and a plain structure: a block
// computes one tile and ends, so the hardware deals the tiles to the CUs as they become free.
// (Persistent blocks with the next tile's loads under way during the epilogue, fragments read
// one sub-step ahead, or half of the waves loading and the other half storing, measured the same or
// slower for the products whose rows are tokens, before their loads were spread over the step: experts
// hold different numbers of rows, and the deal evens that out.  The weight gradients, whose tiles are all alike,
// gain by persistent blocks: gemm_wgrad.hip.)
//
// What bounds it.  With few rows per expert: streaming the weights from HBM.  So a tile is as tall
// as the capacity asks for, every weight line is read once, and rows that do not exist cost no
// traffic (the buffer descriptors end at the kept rows).  With many rows: the L2 -> LDS requests,
// each of which waits for HBM or L2 (the loads of the 256 x 256 tile alone, without products and
// LDS reads, take 85-90 % of the kernel's time).  So the tall tiles are as large as the registers
// allow: eight waves with 3 x 4 or 2 x 5 MFMA tiles of 32 x 32 each hold 256 x 384 or 320 x 256
// accumulators, 20 % fewer operand bytes per product than 256 x 256.
//
// A block has WP x WQ waves, each with 2 IP x 2 IQ MFMA 16x16x32 tiles (P is the MFMA "A" side).  (Of 32x32x16 tiles half
// as many instructions do the same products with the same reads, but they draw more power: with random operands
// and nothing else the chip holds 1750 TFLOP/s with them and 2060 with 16x16x32; beside the loads both run at 2.0-2.2 GHz.)  k advances 64 (BK)
// at a time through STAGES LDS stages filled by direct loads.
#include <math.h>

#include "common.h"
#include "lds_operands.h"
#include "router_wgrad.h"
#include "rows_operands.h"

namespace sw {

constexpr int BK = 64;

struct RowsArgs {
    const bf16 *Q;             // per expert q_batch elements: [rows][ldq], weight gradients [slot][ldq]
    const bf16 *P;             // per expert p_batch elements
    bf16 *Cout;                // per expert c_batch elements, [rows][ldc]
    uint8_t *bits;             // ReLU bits: ROWS_RELU writes, ROWS_MASK reads
    size_t q_batch, p_batch, c_batch;
    int ldq, ldp, ldc;
    int Qdim, Pdim, Kdim;
    const int32_t *kept, *hit;
    int tiles_q, tiles_p, total;
    int E;
    int grid_x;
    int by_xcd;                // an expert's tiles run on one XCD
    const int32_t *slot_token; // dropout, ROWS_COMBINE: token of each slot, [expert][slots]
    const float *slot_gate;    // ROWS_COMBINE: and its gate
    bf16 *y;                   // ROWS_COMBINE: [token][ldc]
    int slots;
    Noise nz;
};

// A skewed router leaves a layer of many experts a handful of tiles, each a CU's work for all of k: up to
// kFewTiles tiles are cut into pieces of 64 x 128, one per block (two experts of 512 tokens, 768 x 3072: forward
// 62 + 97 us -> 36 + 35, data gradients 65 + 107 -> 32 + 31).  Decided by the blocks from the counts, which only the
// device knows; up to 64 kFewExperts experts.
constexpr int kFewExperts = 4, kFewTiles = 64;

// ROWS_COMBINE: the rows, times the gates of their tokens, also go to the tokens' rows of y.
enum { ROWS_PLAIN = 0, ROWS_RELU = 1, ROWS_MASK = 2, ROWS_COMBINE = 3 };

// The tile's products and epilogue, with IQ row blocks of 32 per wave (IQ_MAX of them fit the tile).
// Mask bits: one byte per 16-byte piece of the output (bits 0..3: low halves of its four words, 4..7:
// high halves), [tile][wave][32-row round][pass][lane] in the order the epilogue handles them.
template <int IP, int WP, int IQ, int IQ_MAX, int WQ, int STAGES, bool P_TRANS, int EPI, bool DROP,
          bool WGRAD, bool GUARD = false, bool ONCE = false>
__device__ __forceinline__ void rows_tile(const RowsArgs &a, char *lds, int L, int e, int q0, int p0, int qlim,
                                          int klim, int lane, int wave) {
    constexpr int NW = WP * WQ, PB = 32 * IP * WP, QB = 32 * IQ_MAX * WQ;
    constexpr int kPBytes = PB * BK * 2, kStage = (PB + QB) * BK * 2;
    const int wp = wave % WP, wq = wave / WP;
    const uint32_t lds0 = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) char *)lds;

    typename std::conditional<P_TRANS, RowsTrans<PB, NW, BK, ONCE>, RowsDirect<PB, NW, BK, ONCE>>::type op;
    typename std::conditional<WGRAD, RowsTrans<QB, NW>, RowsDirect<QB, NW>>::type oq;
    op.init_frag16(lane, wp * 32 * IP);
    oq.init_frag16(lane, wq * 32 * IQ);
    op.init(a.P + (size_t)e * a.p_batch, a.ldp, p0, a.Pdim, klim, lane, wave);
    oq.init(a.Q + (size_t)e * a.q_batch, a.ldq, q0, qlim, klim, lane, wave);
    constexpr int kLoadsP = decltype(op)::kLoads;
    constexpr int kLoads = kLoadsP + decltype(oq)::kLoads * IQ / IQ_MAX;   // (load i: rows of block row i and up)
    static_assert(IQ == IQ_MAX || (!WGRAD && decltype(oq)::kLoads == IQ_MAX), "a load per block row");
    const int nk = (klim + BK - 1) / BK;

    // the wave's bits of 32-row round j
    constexpr int kBitBytes = 2 * IP;   // per lane
    auto bits_of = [&](int j) { return a.bits + (((size_t)L * NW + wave) * IQ_MAX + j) * (64 * kBitBytes); };
    uint32_t mb[IQ][2];
    if (EPI == ROWS_MASK) {
#pragma unroll
        for (int j = 0; j < IQ; ++j) {
            const uint8_t *b = bits_of(j);
            mb[j][0] = IP == 1 ? ((const uint16_t *)b)[lane] : ((const uint32_t *)b)[lane];
            mb[j][1] = IP == 3 ? ((const uint16_t *)(b + 256))[lane] : 0u;
        }
    }

    f32x4 acc[2 * IP][2 * IQ];
#pragma unroll
    for (int i = 0; i < 2 * IP; ++i)
#pragma unroll
        for (int j = 0; j < 2 * IQ; ++j) acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};

    auto issue_load = [&](uint32_t at, int kt, int i) {   // load i of a step (past the end: never read)
        if (i < kLoadsP) op.issue_one(at, kt * BK, wave, i);
        else oq.issue_one(at + kPBytes, kt * BK, wave, i - kLoadsP);
    };
    auto issue = [&](int kt, int st) {
#pragma unroll
        for (int i = 0; i < kLoads; ++i) issue_load(lds0 + (uint32_t)(st * kStage), kt, i);
    };
    // Eight waves, two stages.  The P fragments of a half step (32 k) are held in registers, the Q fragments pass by, one
    // ahead.  So P's stage is free once the fragments of its second half are read, in the middle of the step, and is filled
    // with the step after the next from there on, Q's stage at the end: every load has between half a step and one
    // and a half to land.  us, loads of the next step only and a barrier per step / here: 128 experts x 512 x 768 x 3072 first
    // forward 314 / 295, second 280 / 253, masked gradient 312 / 296, first data gradient 283 / 257; 64 x 256 x 4096 x 10240
    // 1346 / 1240, 1327 / 1170, 1470 / 1382, 1434 / 1300.  (The next P fragments read between the products that use the
    // present ones last: registers spill.)
    if constexpr (NW == 8 && STAGES == 2) {
        constexpr int kLoadsQ = kLoads - kLoadsP, kGroups = 2 * IQ;   // groups of products per half step
        auto issue_p = [&](int kt, int i) { issue_load(lds0 + (uint32_t)((kt & 1) * kStage), kt, i); };
        auto issue_q = [&](int kt, int i) { issue_load(lds0 + (uint32_t)((kt & 1) * kStage), kt, kLoadsP + i); };
#pragma unroll
        for (int i = 0; i < kLoads; ++i) issue_load(lds0, 0, i);
#pragma unroll
        for (int i = 0; i < kLoadsP; ++i) issue_p(1, i);
        rows_wait_vmcnt<kLoadsP>();
        __syncthreads();
        bf16x8 held[2 * IP], next = oq.frag16(lds + kPBytes, 0, 0);
#pragma unroll
        for (int i = 0; i < 2 * IP; ++i) held[i] = op.frag16(lds, i, 0);
#pragma nounroll
        for (int kt = 0; kt < nk; ++kt) {
            const char *sp = lds + (kt & 1) * kStage, *sq = sp + kPBytes;
            const char *np = lds + (~kt & 1) * kStage, *nq = np + kPBytes;
#pragma unroll
            for (int ks = 0; ks < 2; ++ks) {
                op.reload_frag();
                oq.reload_frag();
#pragma unroll
                for (int j = 0; j < kGroups; ++j) {
                    const bool last = j == kGroups - 1;
                    const bf16x8 fq = next;
                    if (ks == 0)
#pragma unroll
                        for (int i = 0; i < kLoadsQ; ++i)
                            if (i == j) issue_q(kt + 1, i);
                    if (ks == 1)
#pragma unroll
                        for (int i = 0; i < kLoadsP; ++i)
                            if (1 + i * (kGroups - 1) / kLoadsP == j) issue_p(kt + 2, i);
                    if (ks == 1 && last) {
                        rows_wait_vmcnt<kLoadsP>();   // step kt + 1 has landed
                        __syncthreads();              // ... for all waves, and Q's stage is read
                        next = oq.frag16(nq, 0, 0);
                    } else {
                        next = last ? oq.frag16(sq, 0, 1) : oq.frag16(sq, j + 1, ks);
                    }
                    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
                    for (int i = 0; i < 2 * IP; ++i)
                        acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(held[i], fq, acc[i][j], 0, 0, 0);
                    if (last)
#pragma unroll
                        for (int i = 0; i < 2 * IP; ++i) held[i] = ks == 0 ? op.frag16(sp, i, 1) : op.frag16(np, i, 0);
                    __builtin_amdgcn_sched_barrier(0);
                    if (ks == 1 && j == 0) __syncthreads();   // all waves have read P's stage
                }
            }
        }
    } else {
#pragma unroll
        for (int s = 0; s < STAGES - 1; ++s) issue(s, s);
        int st = 0, fill = STAGES - 1;
        for (int kt = 0; kt < nk; ++kt) {
            if (STAGES == 1) {   // a single stage: other blocks of the CU cover the wait
                if (kt) __syncthreads();
                issue(kt, 0);
            }
            rows_wait_vmcnt<(STAGES > 2 ? STAGES - 2 : 0) * kLoads>();   // step kt has landed
            __syncthreads();                                             // ... for all waves; step kt - 1 is read
            if (STAGES > 1) issue(kt + STAGES - 1, fill);
            const char *sp = lds + st * kStage, *sq = sp + kPBytes;
#pragma unroll
            for (int ks = 0; ks < BK / 32; ++ks) {
                // a half step past an expert's last slot: zeros (us, second gradient with / without these products: 25
                // slots, 104 experts of 2000 x 8032 771 / 720; 4 slots, 128 of 768 x 1536 61 / 57)
                if (WGRAD && kt * BK + ks * 32 >= klim) break;
                bf16x8 fp[2 * IP], fq[2 * IQ];
#pragma unroll
                for (int i = 0; i < 2 * IP; ++i) fp[i] = op.frag16(sp, i, ks);
#pragma unroll
                for (int j = 0; j < 2 * IQ; ++j) fq[j] = oq.frag16(sq, j, ks);
#pragma unroll
                for (int j = 0; j < 2 * IQ; ++j)
#pragma unroll
                    for (int i = 0; i < 2 * IP; ++i)
                        acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(fp[i], fq[j], acc[i][j], 0, 0, 0);
            }
            st = st == STAGES - 1 ? 0 : st + 1;
            fill = fill == STAGES - 1 ? 0 : fill + 1;
        }
    }
    rows_wait_vmcnt<0>();   // the trailing loads
    __syncthreads();

    // Epilogue: 32 rows at a time through LDS of the wave's own, so that rows leave in segments
    // of 32 IP columns, 16 bytes per lane.
    constexpr int kPitch = rows_turn_pitch(IP), kChunks = 4 * IP, kPasses = 2 * IP;
    char *ep = lds + wave * 32 * kPitch;
    const int pw = p0 + wp * 32 * IP;
    auto swz = [](int row) { return IP == 1 ? (row >> 2) & 3 : IP == 2 ? (row >> 1) & 7 : 0; };
    // Stores through a descriptor: rows past the last one and columns past the matrix get an offset outside it
    // and store nothing, without a branch per store.  GUARD: with one, which spaces the stores; large weight gradients of
    // rows that share lines gain by it (see rows_part_lines; us of both gradients, with / without, five tokens per
    // expert, 208 experts of 1080 x 2408 456 / 486, 34 of 2160 x 8520 569 / 588; smaller ones and whole lines lose, 69 of
    // 616 x 1944 73 / 68, 110 of 768 x 3072 193 / 185).
    const auto crsrc = __builtin_amdgcn_make_buffer_rsrc(a.Cout + (size_t)e * a.c_batch, 0,
                                                         (int)((uint32_t)qlim * (uint32_t)a.ldc * 2u), 0x00020000);
    const uint32_t c_step = 64u * (uint32_t)a.ldc;   // bytes of 32 rows
    uint32_t cvoff[kPasses];   // of the lane's piece in pass x, first 32 rows of the wave,
    int left[kPasses];         // and the rows from there to the last one (offsets of rows past it may wrap)
#pragma unroll
    for (int x = 0; x < kPasses; ++x) {
        const int at = x * 64 + lane, row = at / kChunks, p = pw + (at - row * kChunks) * 8;
        cvoff[x] = ((uint32_t)(q0 + wq * IQ * 32 + row) * (uint32_t)a.ldc + (uint32_t)p) * 2u;
        left[x] = p < a.Pdim ? qlim - (q0 + wq * IQ * 32 + row) : 0;
    }
#pragma unroll
    for (int j = 0; j < IQ; ++j) {
        const int qw = q0 + (wq * IQ + j) * 32;
        if (qw >= qlim) break;
#pragma unroll
        for (int h = 0; h < 2; ++h) {   // rows 16 h .. + 15
            const int wrow = 16 * h + (lane & 15);
            // expert dropout: the draw of hidden unit p of token t is element t * d_ff + p
            uint32_t drop_row = 0;
            if (DROP && EPI == ROWS_RELU) {
                const int q = qw + wrow;
                const int tok = q < qlim ? a.slot_token[(size_t)e * a.slots + q] : 0;
                drop_row = (uint32_t)tok * (uint32_t)a.Pdim + (uint32_t)(pw + ((lane >> 4) << 2));
            }
#pragma unroll
            for (int i = 0; i < 2 * IP; ++i) {
                float v[4];
#pragma unroll
                for (int r = 0; r < 4; ++r) v[r] = acc[i][2 * j + h][r];
                if (DROP && EPI == ROWS_RELU) {
                    const uint32_t first = drop_row + (uint32_t)(i * 16);
#pragma unroll
                    for (int m = 0; m < 2; ++m) {
                        const uint32_t z = dropout_pair_bits(a.nz, (first >> 1) + (uint32_t)m);
                        v[2 * m] = dropout_keeps_even(a.nz, z) ? v[2 * m] * a.nz.drop_scale : 0.f;
                        v[2 * m + 1] = dropout_keeps_odd(a.nz, z) ? v[2 * m + 1] * a.nz.drop_scale : 0.f;
                    }
                }
                if (DROP && EPI == ROWS_MASK)
#pragma unroll
                    for (int r = 0; r < 4; ++r) v[r] *= a.nz.drop_scale;
                uint2 o = make_uint2(pack_bf16(v[0], v[1]), pack_bf16(v[2], v[3]));
                if (EPI == ROWS_RELU) {   // on the bf16 values: negative ones (and -0) are < 0 as integers
                    o.x = pk_max_i16(o.x, 0u);
                    o.y = pk_max_i16(o.y, 0u);
                }
                const int ch = i * 2 + (lane >> 5);
                *(uint2 *)(ep + wrow * kPitch + ((ch ^ swz(wrow)) << 4) + ((lane >> 4 & 1) << 3)) = o;
            }
        }
        uint32_t nb[2] = {0u, 0u};
        int tok[kPasses];
        float gate[kPasses];
        if (EPI == ROWS_COMBINE)
#pragma unroll
            for (int x = 0; x < kPasses; ++x) {
                const bool in = 32 * j < left[x];
                const size_t at = (size_t)e * a.slots + (in ? qw + (x * 64 + lane) / kChunks : 0);
                tok[x] = in ? a.slot_token[at] : -1;
                gate[x] = a.slot_gate[at];
            }
#pragma unroll
        for (int x = 0; x < kPasses; ++x) {
            const int at = x * 64 + lane;
            const int row = at / kChunks, c = at - row * kChunks;
            u32x4 val = *(const u32x4 *)(ep + row * kPitch + ((c ^ swz(row)) << 4));
            if (EPI == ROWS_RELU) {   // after ReLU a half word is > 0 exactly when min(., 1) is 1
                uint32_t u = 0;
#pragma unroll
                for (int w = 0; w < 4; ++w) u |= pk_min_u16(val[w], 0x00010001u) << w;
                nb[x >> 2] |= ((u & 0xfu) | ((u >> 12) & 0xf0u)) << (8 * (x & 3));
            }
            if (EPI == ROWS_MASK) {
                uint32_t byte = (mb[j][x >> 2] >> (8 * (x & 3))) & 0xffu;
                byte |= byte << 12;   // bit w -> bit w, bit 4 + w -> bit 16 + w
#pragma unroll
                for (int w = 0; w < 4; ++w) val[w] &= ((byte >> w) & 0x10001u) * 0xffffu;
            }
            const uint32_t off = 32 * j < left[x] ? cvoff[x] + (uint32_t)j * c_step : kOobOffset;
            if (!GUARD || off != kOobOffset) __builtin_amdgcn_raw_buffer_store_b128(val, crsrc, (int)off, 0, 0);
            if (EPI == ROWS_COMBINE && tok[x] >= 0) {   // of the rounded values, as the combine pass
                u32x4 out;
#pragma unroll
                for (int w = 0; w < 4; ++w)
                    out[w] = pack_bf16(__uint_as_float(val[w] << 16) * gate[x],
                                       __uint_as_float(val[w] & 0xffff0000u) * gate[x]);
                *(u32x4 *)(a.y + (size_t)tok[x] * a.ldc + pw + c * 8) = out;
            }
        }
        if (EPI == ROWS_RELU) {
            uint8_t *b = bits_of(j);
            if (IP == 1) ((uint16_t *)b)[lane] = (uint16_t)nb[0];
            else ((uint32_t *)b)[lane] = nb[0];
            if (IP == 3) ((uint16_t *)(b + 256))[lane] = (uint16_t)nb[1];
        }
    }
}

// The wave's share of the tile's rows comes in IQ blocks of 32.  Tiles of eight waves that hold fewer rows run
// with as few blocks as hold them, so with fewer products, fragment reads and loads (128 experts of 768 x 3072, 64
// rows in tiles of 256: masked gradient 152 -> 140 us, first forward 186 -> 176; 64 of 4096 x 10240, 256 rows in
// tiles of 320: 1530 -> 1480).
template <int IP, int WP, int IQ, int WQ, int STAGES, bool P_TRANS, int EPI, bool DROP, bool WGRAD, bool GUARD = false,
          bool ONCE = false>
__device__ __forceinline__ void rows_block(const RowsArgs &a, char *lds, int L) {
    constexpr int PB = 32 * IP * WP, QB = 32 * IQ * WQ;
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
    if constexpr (WP * WQ == 8 && !WGRAD) {
        if (a.E <= 64 * kFewExperts && *a.hit * a.tiles_p <= kFewTiles) {
            constexpr int kSubRows = QB / 64, kSubs = kSubRows * (PB / 128);
            // row tiles of experts lane, lane + 64, .. (more than the limit: one more than it, so that their sum is
            // right up to the limit and above it beyond)
            int rows[kFewExperts], tiles = 0;
#pragma unroll
            for (int m = 0; m < kFewExperts; ++m) {
                rows[m] = lane + 64 * m < a.E ? min((min(a.kept[lane + 64 * m], a.Qdim) + QB - 1) / QB, kFewTiles + 1) : 0;
#pragma unroll
                for (int b = 0; (kFewTiles + 1) >> b; ++b)   // a digit at a time
                    tiles += __popcll(__ballot(rows[m] >> b & 1)) << b;
            }
            tiles *= a.tiles_p;
            if (tiles > 0 && tiles <= kFewTiles && tiles * kSubs <= a.total) {
                int at = L / kSubs, sub = L - at * kSubs, e = 0;
                if (at >= tiles) return;
#pragma unroll
                for (int m = 0; m < kFewExperts; ++m)
                    for (int i = 0; i < 64; ++i) {
                        const int n = __builtin_amdgcn_readlane(rows[m], i) * a.tiles_p;
                        if (at < n) {
                            e = 64 * m + i;
                            const int tq = n / a.tiles_p, pt = at / tq;
                            const int qlim = min(a.kept[e], a.Qdim);
                            const int q0 = (at - pt * tq) * QB + sub % kSubRows * 64, p0 = pt * PB + sub / kSubRows * 128;
                            if (q0 < qlim && p0 < a.Pdim)
                                rows_tile<1, 4, 1, 1, 2, (STAGES * (PB + QB)) / 192, P_TRANS, EPI, DROP, false>(
                                    a, lds, L, e, q0, p0, qlim, a.Kdim, lane, wave);
                            return;
                        }
                        at -= n;
                    }
                return;
            }
        }
    }
    if (a.by_xcd) {   // block b runs on XCD b mod 8: give each XCD a range of experts
        const int per = (a.total + 7) >> 3, at = L >> 3;
        L = (L & 7) * per + at;
        if (at >= per) return;
    }
    if (L >= a.total) return;
    const int per_e = a.tiles_p * a.tiles_q;
    const int e = L / per_e, rem = L - e * per_e;
    int pt, qt;   // the dimension with fewer tiles runs fastest: sharers of the larger operand are neighbours
    if (a.tiles_q <= a.tiles_p) {
        pt = rem / a.tiles_q;
        qt = rem - pt * a.tiles_q;
    } else {
        qt = rem / a.tiles_p;
        pt = rem - qt * a.tiles_p;
    }
    const int used = a.kept[e];   // slots with a token
    const int qlim = WGRAD ? a.Qdim : min(used, a.Qdim), klim = WGRAD ? min(used, a.Kdim) : a.Kdim;
    const int q0 = qt * QB, p0 = pt * PB;
    if (q0 >= qlim) return;
#define SW_ROWS(N) \
    rows_tile<IP, WP, (N) < IQ ? (N) : IQ, IQ, WQ, STAGES, P_TRANS, EPI, DROP, WGRAD, GUARD, ONCE>( \
        a, lds, L, e, q0, p0, qlim, klim, lane, wave)
    if constexpr (WP * WQ == 8 && !WGRAD) {
        const int blocks = (qlim - q0 + 32 * WQ - 1) / (32 * WQ);
        if (blocks <= 1) SW_ROWS(1);
        else if (blocks == 2) SW_ROWS(2);
        else if (blocks == 3) SW_ROWS(3);
        else if (blocks == 4 || IQ == 4) SW_ROWS(4);
        else if constexpr (IQ > 4) SW_ROWS(5);
    } else {
        SW_ROWS(IQ);
    }
#undef SW_ROWS
}

template <int IP, int WP, int IQ, int WQ, int STAGES, int WPE, bool P_TRANS, int EPI, bool DROP,
          bool ONCE, bool WGRAD, bool GUARD>
__global__ __launch_bounds__(64 * WP * WQ, WPE) void gemm_rows_kernel(RowsArgs a) {
    extern __shared__ __attribute__((aligned(16))) char lds[];
    rows_block<IP, WP, IQ, WQ, STAGES, P_TRANS, EPI, DROP, WGRAD, GUARD, ONCE>(a, lds,
                                                                               blockIdx.y * a.grid_x + blockIdx.x);
}

// Three products in one launch: the first layer's data gradient and both weight gradients, which do not depend on
// each other.  Tiles of four waves.
struct RowsArgs3 {
    RowsArgs data, first, second;
    int end[3];   // blocks up to the end of the data gradient and of each weight gradient (multiples of eight)
    RouterWgradArgs router;   // parts of the router's weight gradient, in blocks behind them
};
template <int IP, int WP, int IQ, int WQ, int STAGES, int GP, int GWP, int GQ, int GWQ, int GSTAGES>
__global__ __launch_bounds__(256, 2) void gemm_rows_backward_kernel(RowsArgs3 a) {
    static_assert(WP * WQ == 4 && GWP * GWQ == 4, "256 threads");
    extern __shared__ __attribute__((aligned(16))) char lds[];
    const int L = blockIdx.x;
    if (L < a.end[0]) rows_block<IP, WP, IQ, WQ, STAGES, false, ROWS_PLAIN, false, false>(a.data, lds, L);
    else if (L < a.end[1])
        rows_block<GP, GWP, GQ, GWQ, GSTAGES, true, ROWS_PLAIN, false, true>(a.first, lds, L - a.end[0]);
    else if (L < a.end[2])
        rows_block<GP, GWP, GQ, GWQ, GSTAGES, true, ROWS_PLAIN, false, true>(a.second, lds, L - a.end[1]);
    else
        router_wgrad_block<bf16>(a.router, L - a.end[2], lds);
}

constexpr int rows_lds(int IP, int WP, int IQ, int WQ, int STAGES) {
    const int ring = STAGES * 32 * (IP * WP + IQ * WQ) * BK * 2, turn = WP * WQ * 32 * rows_turn_pitch(IP);
    return ring > turn ? ring : turn;
}

// sets the tile counts; returns the blocks to launch
static int64_t rows_plan(RowsArgs &a, int E, int QB, int PB, bool wgrad) {
    a.tiles_q = (int)ceil_div(a.Qdim, QB);
    a.tiles_p = (int)ceil_div(a.Pdim, PB);
    a.total = a.tiles_q * a.tiles_p * E;
    a.E = E;
    // Up to 64 rows the shared operand is small next to the weights: the tiles are dealt over all XCDs
    // in order, which stays even when only some experts hold tokens.
    a.by_xcd = wgrad || QB > 64;
    return a.by_xcd ? ceil_div(a.total, 8) * 8 : a.total;
}

template <int IP, int WP, int IQ, int WQ, int STAGES, int WPE, bool P_TRANS, int EPI, bool DROP,
          bool ONCE, bool WGRAD, bool GUARD = false>
static hipError_t rows_launch(RowsArgs a, int E, hipStream_t s) {
    auto kern = gemm_rows_kernel<IP, WP, IQ, WQ, STAGES, WPE, P_TRANS, EPI, DROP, ONCE, WGRAD, GUARD>;
    constexpr int PB = 32 * IP * WP, QB = 32 * IQ * WQ;
    constexpr int lds = rows_lds(IP, WP, IQ, WQ, STAGES);
    static PerDeviceOnce once;
    hipError_t err = once_per_device(once, [&] {
        return hipFuncSetAttribute((const void *)kern, hipFuncAttributeMaxDynamicSharedMemorySize, lds);
    });
    if (err != hipSuccess) return err;
    const int64_t blocks = rows_plan(a, E, QB, PB, WGRAD);
    const int64_t most = kMaxGridThreads / (64 * WP * WQ) / 8 * 8;   // (whole rounds of XCDs)
    a.grid_x = (int)(blocks < most ? blocks : most);
    hipLaunchKernelGGL(kern, dim3((unsigned)a.grid_x, (unsigned)ceil_div(blocks, a.grid_x)), dim3(64 * WP * WQ), lds,
                       s, a);
    return hipGetLastError();
}

// ---- which tile ---------------------------------------------------------------------
// Per tile shape: CU time of one 64-k step and of a tile's start and epilogue (microseconds, all
// CUs busy), and the rate at which the shape streams weights when they are what it waits for
// (GB/s).  Measured on 128 experts of 768 x 3072 with 16 .. 512 rows each, when a tile cost the same however
// many rows it held; the estimate made from them picked the fastest or one within 5 % of it over that range
// and at 64 experts of 4096 x 10240.  Since then tiles of eight waves with few rows run with fewer row blocks,
// which only 256 x 384's line below knows of, and have their loads further ahead (6-12 % less per step, not measured
// again here): between 64 and 200 rows per expert, and where 256 x 256 wins by a few per cent, the choice may be off
// by more.
struct RowsModel {
    int tile, qb, pb;
    double step, once, gbs;
};
static const RowsModel kRowsModels[] = {
    {ROWS_32x128, 32, 128, 0.52, 1.4, 5300.},  {ROWS_64x256, 64, 256, 1.30, 2.2, 5300.},
    {ROWS_96x128, 96, 128, 0.66, 1.4, 4100.},  {ROWS_128x128, 128, 128, 0.65, 1.4, 4000.},
    {ROWS_256x256, 256, 256, 2.10, 2.5, 3800.}, {ROWS_320x256, 320, 256, 2.20, 3.5, 3800.},
    {ROWS_256x384, 256, 384, 2.86, 5.0, 4850.},
};

// Tiles of qb rows an expert takes on average: counts scatter around the mean by the routing's own
// spread (about an eighth of it, from the router's initialisation) and by chance.
static double rows_tiles(double mean, double cap, int qb) {
    const double sd = sqrt(mean + 0.0169 * mean * mean);
    static const double at[5] = {-1.3, -0.5, 0.0, 0.5, 1.3};
    double sum = 0.;
    for (double x : at) {
        double c = mean + sd * x;
        c = c < 1. ? 1. : (c > cap ? cap : c);
        sum += ceil(c / qb);
    }
    return sum / 5.;
}

bool rows_count_hit(const Workspace &w) {
    for (GemmKind k : {GEMM_FWD1, GEMM_FWD2, GEMM_DGRAD2, GEMM_DGRAD1})   // (tiles of eight waves: rows_block)
        if (w.gemm_tile[k] >= ROWS_256x256) return w.E <= 64 * kFewExperts;
    return false;
}

int64_t rows_bits_bytes(int tile, int64_t E, int64_t C, int64_t f) {
    for (const RowsModel &m : kRowsModels)
        if (m.tile == tile) return E * ceil_div(C, m.qb) * ceil_div(f, m.pb) * (m.qb * m.pb / 8);
    return 0;
}

// Tile of a row-limited product of Pdim columns over Kdim.
int rows_tile_for(const Workspace &w, int64_t Pdim, int64_t Kdim, int64_t bits_limit) {
    if (w.C == 0) return ROWS_256x256;   // nothing will be launched
    const double cap = (double)w.C, mean = fmin((double)w.T / (double)w.E, cap);
    const double steps = ceil(Kdim / 64.);
    // experts that get a token at all
    const double hit = (double)w.E * (1. - pow(1. - 1. / (double)w.E, (double)w.T));
    int best = ROWS_256x256;
    double best_us = 1e30;
    for (const RowsModel &m : kRowsModels) {
        if (rows_bits_bytes(m.tile, w.E, w.C, Pdim) > bits_limit) continue;   // (never 256 x 256)
        const double tq = rows_tiles(mean, cap, m.qb);
        const double tiles = hit * tq * ceil((double)Pdim / m.pb);
        // an expert's second tile finds the weights in L2 if it runs on the same XCD
        const double reads = m.qb > 64 ? 1. : tq;
        const double bytes = hit * (reads * Pdim * Kdim + mean * (Pdim + Kdim)) * 2.;
        // rows that do not exist are not loaded; the widest tile, which waits for its loads most, gains by it,
        // down to the time of its products at the sustained MFMA rate (1.5 us for all of its rows).  Without that
        // limit it was taken for a handful of rows of a shallow layer: 8 rows, 256 experts of 264 x 2704, masked
        // gradient 123 us, with 32 x 128 tiles 83.
        const double fill = mean / (tq * m.qb);
        const double step = m.tile == ROWS_256x384 ? fmax(m.step * fmin(0.36 + 0.75 * fill, 1.), 1.5) : m.step;
        // (fewer tiles than CUs: the longest block is the time)
        const double us = fmax((steps * step + m.once) * fmax(tiles / 256., 1.), bytes / m.gbs * 1e-3);
        if (us < best_us * 0.97) {   // later, larger tiles have to be clearly better
            best = m.tile;
            best_us = us;
        }
    }
    return best;
}

// Weight gradients: CU time of a 64-k step and of a tile's epilogue (and start) per shape; persistent blocks
// take whole rounds.  Fitted to 22 shapes of 4 .. 256 experts, 64 .. 4096 wide, 4 .. 7500 slots; us of the first
// gradient measured, estimated best first (256 x 384 or 384 x 256: gemm_wgrad.hip; 256 x 256: gemm_bf16.hip):
//   128 experts of 768 x 3072, 512 slots   384x256 299, 256x128 326, 256x256 334
//   32 of 512 x 1024, 1024 slots           256x256 37, 256x384 41, 256x128 41, 128x128 51
//   32 of 512 x 1024, 256 slots            256x128 16, 128x128 17, 256x384 18, 256x256 18
//   16 of 128 x 512, 3750 slots            128x128 38, 256x256 73, 256x128 76, 256x384 97
struct WgradModel {
    int tile, qb, pb;
    double step, once;
    bool rounds;
};
static const WgradModel kWgradModels[] = {
    {ROWS_128x128, 128, 128, 0.65, 1.4, false}, {ROWS_256x128, 256, 128, 0.95, 2.2, false},
    {ROWS_NONE, 256, 256, 1.5, 6.0, true},      {ROWS_256x384, 256, 384, 2.05, 6.0, true},
    {ROWS_384x256, 384, 256, 2.05, 6.0, true},
};

// A weight gradient whose rows begin inside a 128-byte line and that is more than twice the memory-side cache: two waves
// write each row's shared lines, and parts of a line that do not meet in L2 go to HBM one by one.
static bool rows_part_lines(const Workspace &w, int64_t Qdim, int64_t Pdim) {
    return Pdim % 64 != 0 && (double)w.E * (double)Qdim * (double)Pdim * 2. > 512e6;
}

// Tile of a weight gradient of Qdim x Pdim; ROWS_NONE: the persistent kernel of gemm_bf16.hip.
int rows_wgrad_tile(const Workspace &w, int64_t Qdim, int64_t Pdim) {
    const double cap = (double)w.C, mean = fmin((double)w.T / (double)w.E, cap);
    // Fewer than eight tokens per expert: little but the store, where two small blocks per CU do as well or better
    // (169 experts of 272 x 2064, 186 tokens: 31 us, 384 x 256 36; 236 of 2000 x 856, 205 tokens: 191, 256 x 384 200;
    // 147 of 296 x 2464, 96 tokens: 43, 128 x 128 48).
    // Large gradients with shared lines: fewer than 32 where the column tiles, which share them, follow each other (us of
    // the second gradient, 256 x 128 / persistent; 208 experts of 1080 x 2408, 12, 24 and 40 tokens each 237 / 271,
    // 255 / 275, 284 / 261; 34 of 2160 x 8520 282 / 336, 288 / 329, 301 / 311; the other way, 32 of 3000 x 6008 with 12
    // tokens each, 406 / 298).
    const bool in_turn = ceil_div(Qdim, 256) > ceil_div(Pdim, 128);
    if (mean < (in_turn && rows_part_lines(w, Qdim, Pdim) ? 32. : 8.))
        return w.E * ceil_div(Qdim, 256) * ceil_div(Pdim, 256) < 256 ? ROWS_128x128 : ROWS_256x128;
    const double steps = rows_tiles(mean, cap, 64);
    int best = ROWS_128x128;
    double best_us = 1e30;
    for (const WgradModel &m : kWgradModels) {
        const double per_cu = (double)(w.E * ceil_div(Qdim, m.qb) * ceil_div(Pdim, m.pb)) / 256.;
        double us = (m.rounds ? ceil(per_cu) : fmax(per_cu, 1.)) * (steps * m.step + m.once);
        // of the two large shapes the one with the long side along the smaller dimension: 64 experts of
        // 4096 x 10240, 256 slots: first gradient 1990 us, second 1980; the other way 2140 and 2080
        if ((m.tile == ROWS_256x384 && Qdim < Pdim) || (m.tile == ROWS_384x256 && Pdim < Qdim)) us *= 1.03;
        if (us < best_us) {
            best = m.tile;
            best_us = us;
        }
    }
    return best;
}

// Weights that no other block reads (one row tile per expert, whole lines) of a layer beyond the memory-side cache
// bypass L2 (nt): they stream faster, and what the cache holds from before, the last gradients written among it, is not
// pushed out to HBM meanwhile.  us of a pass, without / with: 64 tokens, 128 experts of 768 x 3072 forward 118.5 / 107.5,
// 2048 267 / 252, 16384 349 / 322, forward + backward 8192 914 / 875; 32 experts (302 MB), 512 tokens forward
// 84 / 81, both 265 / 241; but 16 experts, which the cache holds, 50 / 61 and 122 / 135; lines shared by tiles, 104
// experts of 2000 x 8032 4570 / 5118; two row tiles, Switch-Base 2008 / 2055.  (320 x 256, 64 experts of 4096 x 10240:
// 9580 / 9575.)
static bool rows_read_once(const Workspace &w, const RowsArgs &a, int QB) {
    return a.Qdim <= QB && a.ldp % 64 == 0 && (double)w.E * (double)w.d * (double)(w.f1 + w.f) * 2. > 256e6;
}

template <int IP, int WP, int IQ, int WQ, int STAGES, bool P_TRANS, int EPI, bool DROP>
static hipError_t rows_stream(const Workspace &w, const RowsArgs &a, hipStream_t s) {
    if (rows_read_once(w, a, 32 * IQ * WQ))
        return rows_launch<IP, WP, IQ, WQ, STAGES, 2, P_TRANS, EPI, DROP, true, false>(a, (int)w.E, s);
    return rows_launch<IP, WP, IQ, WQ, STAGES, 2, P_TRANS, EPI, DROP, false, false>(a, (int)w.E, s);
}

template <bool P_TRANS, int EPI, bool DROP>
static hipError_t rows_by_tile(const Workspace &w, const RowsArgs &a, int tile, hipStream_t s) {
    switch (tile) {
    case ROWS_32x128: return rows_stream<1, 4, 1, 1, 3, P_TRANS, EPI, DROP>(w, a, s);
    case ROWS_64x256: return rows_stream<2, 4, 2, 1, 2, P_TRANS, EPI, DROP>(w, a, s);
    case ROWS_96x128: return rows_stream<1, 4, 3, 1, 2, P_TRANS, EPI, DROP>(w, a, s);
    case ROWS_128x128: return rows_stream<2, 2, 2, 2, 2, P_TRANS, EPI, DROP>(w, a, s);
    }
    if constexpr (EPI != ROWS_COMBINE) switch (tile) {
    case ROWS_256x256: return rows_launch<2, 4, 4, 2, 2, 2, P_TRANS, EPI, DROP, false, false>(a, (int)w.E, s);
    case ROWS_320x256: return rows_launch<2, 4, 5, 2, 2, 2, P_TRANS, EPI, DROP, false, false>(a, (int)w.E, s);
    case ROWS_256x384: return rows_stream<3, 4, 4, 2, 2, P_TRANS, EPI, DROP>(w, a, s);
    }
    return hipErrorInvalidValue;
}

// Operands and output of a product.
static RowsArgs rows_args(GemmKind kind, const Workspace &w, char *ws, const void *W_in, const void *W_out,
                          void *dW_in, void *dW_out) {
    const int d = (int)w.d, f = (int)w.f, f1 = (int)w.f1, C = (int)w.C;
    RowsArgs a{};
    a.kept = (const int32_t *)(ws + w.kept);
    a.hit = (const int32_t *)(ws + w.hit);
    a.slot_token = (const int32_t *)(ws + w.slot_token);
    a.slots = C;
    a.nz = w.noise;
    a.bits = (uint8_t *)(ws + w.relu_bits);
    auto set = [&](size_t q, int ldq, const void *P, size_t p_batch, int ldp, size_t c, int ldc) {
        a.Q = (const bf16 *)(ws + q); a.q_batch = (size_t)C * ldq; a.ldq = ldq;
        a.P = (const bf16 *)P; a.p_batch = p_batch; a.ldp = ldp;
        a.Cout = (bf16 *)(ws + c); a.c_batch = (size_t)C * ldc; a.ldc = ldc;
        a.Qdim = C; a.Pdim = ldc; a.Kdim = ldq;
    };
    auto set_wgrad = [&](size_t q, int ldq, size_t p, int ldp, void *out) {
        a.Q = (const bf16 *)(ws + q); a.q_batch = (size_t)C * ldq; a.ldq = ldq;
        a.P = (const bf16 *)(ws + p); a.p_batch = (size_t)C * ldp; a.ldp = ldp;
        a.Cout = (bf16 *)out; a.c_batch = (size_t)ldq * ldp; a.ldc = ldp;
        a.Qdim = ldq; a.Pdim = ldp; a.Kdim = C;
    };
    switch (kind) {
    case GEMM_FWD1: set(w.Xd, d, W_in, (size_t)d * f1, f1, w.geglu ? w.H : w.A, f1); break;
    case GEMM_FWD2: set(w.A, f, W_out, (size_t)f * d, d, w.O, d); break;
    case GEMM_DGRAD2: set(w.dO, d, W_out, (size_t)f * d, d, w.geglu ? w.dA : w.dH, f); break;
    case GEMM_DGRAD1: set(w.dH, f1, W_in, (size_t)d * f1, f1, w.dXd, d); break;
    case GEMM_WGRAD2: set_wgrad(w.A, f, w.dO, d, dW_out); break;
    case GEMM_WGRAD1: set_wgrad(w.Xd, d, w.dH, f1, dW_in); break;
    }
    return a;
}

hipError_t launch_gemm_rows(GemmKind kind, const Workspace &w, char *ws, const void *W_in, const void *W_out,
                            void *dW_in, void *dW_out, void *y, int tile, hipStream_t s) {
    const int C = (int)w.C, E = (int)w.E;
    RowsArgs a = rows_args(kind, w, ws, W_in, W_out, dW_in, dW_out);
    a.slot_gate = (const float *)(ws + w.slot_gate);
    a.y = (bf16 *)y;
    const bool drop = w.noise.dropout;
    if (C == 0 && kind != GEMM_WGRAD1 && kind != GEMM_WGRAD2) return hipSuccess;
    switch (kind) {
    case GEMM_FWD1: {
        ProfScope ps(w.geglu ? "gemm1_fwd" : "gemm1_fwd_relu", s);
        if (w.geglu) return rows_by_tile<true, ROWS_PLAIN, false>(w, a, tile, s);
        if (drop) return rows_by_tile<true, ROWS_RELU, true>(w, a, tile, s);
        return rows_by_tile<true, ROWS_RELU, false>(w, a, tile, s);
    }
    case GEMM_FWD2: {
        ProfScope ps("gemm2_fwd", s);
        if (w.combine_in_gemm) return rows_by_tile<true, ROWS_COMBINE, false>(w, a, tile, s);
        return rows_by_tile<true, ROWS_PLAIN, false>(w, a, tile, s);
    }
    case GEMM_DGRAD2: {
        ProfScope ps(w.geglu ? "gemm2_dgrad" : "gemm2_dgrad_relumask", s);
        if (w.geglu) return rows_by_tile<false, ROWS_PLAIN, false>(w, a, tile, s);
        if (drop) return rows_by_tile<false, ROWS_MASK, true>(w, a, tile, s);
        return rows_by_tile<false, ROWS_MASK, false>(w, a, tile, s);
    }
    case GEMM_DGRAD1: {
        ProfScope ps("gemm1_dgrad", s);
        return rows_by_tile<false, ROWS_PLAIN, false>(w, a, tile, s);
    }
    case GEMM_WGRAD2:
    case GEMM_WGRAD1: {
        if (tile == ROWS_256x384 || tile == ROWS_384x256) return launch_gemm_wgrad(kind, w, ws, dW_in, dW_out, tile, s);
        const bool two = kind == GEMM_WGRAD2;
        ProfScope ps(two ? "gemm2_wgrad" : "gemm1_wgrad", s);
        switch (tile) {
        case ROWS_128x128: return rows_launch<2, 2, 2, 2, 2, 2, true, ROWS_PLAIN, false, false, true>(a, E, s);
        case ROWS_256x128: {
            // Three blocks per CU, which 168 registers allow, cover the waits of a single stage where an expert has more than
            // one step of slots; with one step the stores bound it and 174 registers are better (us of both gradients, two /
            // three: 39584 x 752 x 2696, 8 experts 592 / 375; of a pass: 512 x 1080 x 2408, 208 experts 1346 / 1388, 64 x 4096 x
            // 1024, 128 experts 780 / 790).
            const bool part = rows_part_lines(w, a.Qdim, a.Pdim);
            if (w.C > BK && w.T > w.E * BK)
                return part ? rows_launch<2, 2, 4, 2, 1, 3, true, ROWS_PLAIN, false, false, true, true>(a, E, s)
                            : rows_launch<2, 2, 4, 2, 1, 3, true, ROWS_PLAIN, false, false, true>(a, E, s);
            return part ? rows_launch<2, 2, 4, 2, 1, 2, true, ROWS_PLAIN, false, false, true, true>(a, E, s)
                        : rows_launch<2, 2, 4, 2, 1, 2, true, ROWS_PLAIN, false, false, true>(a, E, s);
        }
        }
        return hipErrorInvalidValue;
    }
    }
    return hipErrorInvalidValue;
}

template <int IP, int WP, int IQ, int WQ, int STAGES, int GP, int GWP, int GQ, int GWQ, int GSTAGES>
static hipError_t rows_backward_launch(RowsArgs3 a, int E, hipStream_t s) {
    auto kern = gemm_rows_backward_kernel<IP, WP, IQ, WQ, STAGES, GP, GWP, GQ, GWQ, GSTAGES>;
    constexpr int l0 = rows_lds(IP, WP, IQ, WQ, STAGES), l1 = rows_lds(GP, GWP, GQ, GWQ, GSTAGES);
    constexpr int lds = l0 > l1 ? l0 : l1;
    static_assert(lds >= kRwLds, "room for the router's blocks");
    static PerDeviceOnce once;
    hipError_t err = once_per_device(once, [&] {
        return hipFuncSetAttribute((const void *)kern, hipFuncAttributeMaxDynamicSharedMemorySize, lds);
    });
    if (err != hipSuccess) return err;
    const int64_t n0 = ceil_div(rows_plan(a.data, E, 32 * IQ * WQ, 32 * IP * WP, false), 8) * 8;
    const int64_t n1 = rows_plan(a.first, E, 32 * GQ * GWQ, 32 * GP * GWP, true);
    const int64_t n2 = rows_plan(a.second, E, 32 * GQ * GWQ, 32 * GP * GWP, true);
    a.end[0] = (int)n0;
    a.end[1] = (int)(n0 + n1);
    a.end[2] = (int)(n0 + n1 + n2);
    hipLaunchKernelGGL(kern, dim3((unsigned)(a.end[2] + a.router.blocks)), dim3(256), lds, s, a);
    return hipGetLastError();
}

// Where the tiles of all three have four waves and the weights are small enough for the memory-side cache: there a
// launch is a good part of a product, and few tiles leave CUs idle at the end of each (us per forward + backward
// pass, three launches / one: 5003 x 392 x 1000, 10 experts 119 / 109; 256 x 64 x 256, 4 experts 53 / 47; 4096 x 256 x 1024,
// 64 experts 120 / 108).  Beyond it the streams of the three disturb each other (512 x 768 x 3072, 128 experts:
// 764 / 778).
bool rows_backward_supported(const Workspace &w) {
    const int t = w.gemm_tile[GEMM_DGRAD1], g = w.gemm_tile[GEMM_WGRAD1];
    return w.C > 0 && !w.fused && t >= ROWS_32x128 && t <= ROWS_128x128 && (g == ROWS_128x128 || g == ROWS_256x128) &&
           w.gemm_tile[GEMM_WGRAD2] == g && (double)w.E * (double)w.d * (double)(w.f1 + w.f) * 2. <= 256e6 &&
           w.E * (ceil_div(w.C, 32) * ceil_div(w.d, 128) + 2 * ceil_div(w.d, 128) * ceil_div(w.f1, 128)) < 1 << 22;
}

hipError_t launch_rows_backward(const Workspace &w, char *ws, const void *W_in, const void *W_out, void *dW_in,
                                void *dW_out, const RouterWgradArgs &parts, hipStream_t s) {
    ProfScope ps("gemm_backward", s);
    RowsArgs3 a{};
    a.router = parts;
    a.data = rows_args(GEMM_DGRAD1, w, ws, W_in, W_out, dW_in, dW_out);
    a.first = rows_args(GEMM_WGRAD1, w, ws, W_in, W_out, dW_in, dW_out);
    a.second = rows_args(GEMM_WGRAD2, w, ws, W_in, W_out, dW_in, dW_out);
    const int E = (int)w.E;
    const bool small = w.gemm_tile[GEMM_WGRAD1] == ROWS_128x128;
    switch (w.gemm_tile[GEMM_DGRAD1]) {
#define SW_THREE(...)                                                             \
    return small ? rows_backward_launch<__VA_ARGS__, 2, 2, 2, 2, 2>(a, E, s)      \
                 : rows_backward_launch<__VA_ARGS__, 2, 2, 4, 2, 1>(a, E, s)
    case ROWS_32x128: SW_THREE(1, 4, 1, 1, 3);
    case ROWS_64x256: SW_THREE(2, 4, 2, 1, 2);
    case ROWS_96x128: SW_THREE(1, 4, 3, 1, 2);
    case ROWS_128x128: SW_THREE(2, 2, 2, 2, 2);
#undef SW_THREE
    }
    return hipErrorInvalidValue;
}

}  // namespace sw
