// Operand tiles of gemm_rows.hip, gemm_wgrad.hip, gemm_f32.hip and router_block.hip: R rows by a step's k, filled by
// NW waves with direct global -> LDS loads.  In a step that the end of k cuts, k past the end reads as zeros; of a
// step wholly past it, which is loaded to keep the wait counts even and never read, nothing is said (its 32-bit
// offsets may wrap back into the descriptor).
#pragma once
#include "lds_operands.h"

namespace sw {

// [row][k] operand of R rows, BK (64 or 32) k per step: LDS [R][BK k]; the 16-byte chunks of a
// row are permuted as in DirectOperand64 / DirectOperand.
template <int R, int NW, int BK = 64, bool ONCE = false> struct RowsDirect {
    static constexpr int kRowsPerLoad = 512 / BK;            // rows of one wave-wide load
    static constexpr int kLoads = R / (kRowsPerLoad * NW);   // per wave and step
    static constexpr int kPitch = BK * 2;                    // bytes of an LDS row
    static_assert(kLoads * kRowsPerLoad * NW == R, "rows divide over the waves");
    static __device__ __forceinline__ int perm(int r) { return BK == 64 ? (r >> 1) & 7 : dswz(r); }
    i32x4 rsrc;
    uint32_t voff, row_step;
    int c8, klim;
    uint32_t frag0;
    __device__ __forceinline__ void init(const bf16 *base, int ld, int row0, int rowlim, int klim_,
                                         int lane, int wave) {
        rsrc = make_rsrc(base, (uint32_t)rowlim * (uint32_t)ld * 2u);
        const int r = wave * kRowsPerLoad + lane / (BK / 8);
        const int c = (lane % (BK / 8)) ^ perm(r);
        c8 = c << 3;
        voff = ((uint32_t)(row0 + r) * (uint32_t)ld + (uint32_t)c8) * 2u;
        row_step = (uint32_t)(kRowsPerLoad * NW) * (uint32_t)ld * 2u;
        klim = klim_;
    }
    __device__ __forceinline__ void init_frag(int lane, int frag_row) {
        const int fr = frag_row + (lane & 31);
        frag0 = (uint32_t)(fr * kPitch + (((lane >> 5) ^ perm(fr)) << 4));
    }
    __device__ __forceinline__ void issue_one(uint32_t st, int k0, int wave, int i) const {
        // (chunks past the last k: the sign of the difference, which is kOobOffset)
        const uint32_t vo = voff | ((uint32_t)(klim - k0 - 1 - c8) & kOobOffset);
        dma16<ONCE>(rsrc, vo, (uint32_t)i * row_step + (uint32_t)k0 * 2u,
              st + (uint32_t)((i * NW + wave) * 1024));
    }
    __device__ __forceinline__ bf16x8 frag(const char *st, int x, int ks) const {
        return *(const bf16x8 *)(st + ((frag0 ^ (uint32_t)(ks << 5)) + (uint32_t)(x * 32 * kPitch)));
    }
    // the same for MFMA 16x16x32: 16 rows, 32 k
    __device__ __forceinline__ void init_frag16(int lane, int frag_row) {
        static_assert(BK == 64, "");
        const int fr = frag_row + (lane & 15);
        frag0 = (uint32_t)(fr * kPitch + (((lane >> 4) ^ perm(fr)) << 4));
    }
    __device__ __forceinline__ void reload_frag() { asm volatile("" : "+v"(frag0)); }   // (see RowsTrans)
    __device__ __forceinline__ bf16x8 frag16(const char *st, int x, int ks) const {
        // (16 rows further the permutation is the same)
        return *(const bf16x8 *)(st + ((frag0 ^ (uint32_t)(ks << 6)) + (uint32_t)(x * 16 * kPitch)));
    }
};

typedef float f32x4 __attribute__((ext_vector_type(4)));

// fp32 [row][k] operand of MFMA tiles of S rows: 32 k = 128 bytes per row, exactly the bf16 layout of 64 k
// (sizes in half words)
template <int R, int NW, int S = 32> struct F32Direct : RowsDirect<R, NW, 64> {
    __device__ __forceinline__ void init(const float *base, int ld, int row0, int rowlim, int klim,
                                         int lane, int wave) {
        RowsDirect<R, NW, 64>::init((const bf16 *)base, 2 * ld, row0, rowlim, 2 * klim, lane, wave);
    }
    __device__ __forceinline__ void issue_one(uint32_t st, int k0, int wave, int i) const {
        RowsDirect<R, NW, 64>::issue_one(st, 2 * k0, wave, i);
    }
    __device__ __forceinline__ void init_frag(int lane, int frag_row) {
        RowsDirect<R, NW, 64>::init_frag(lane % S, frag_row);   // all parts of the wave: chunk 2 ks ...
        part = lane / S;
    }
    // element m: k = 8 ks + 64 / S m + lane / S (... and chunk 2 ks + 1)
    __device__ __forceinline__ f32x4 frag4(const char *st, int x, int ks) const {
        const char *p = st + (uint32_t)(x * 32 * 128);
        const uint32_t at = this->frag0 ^ (uint32_t)(ks << 5);
        if (S == 16)
            return f32x4{*(const float *)(p + at + 4 * part), *(const float *)(p + (at ^ 16u) + 4 * part), 0.f, 0.f};
        const f32x4 a = *(const f32x4 *)(p + at), b = *(const f32x4 *)(p + (at ^ 16u));
        return part ? f32x4{a[1], a[3], b[1], b[3]} : f32x4{a[0], a[2], b[0], b[2]};
    }
    int part;
};

// [k][row] operand of R rows for MFMA 16x16x32: LDS [64 k][R].  One transposing read (ds_read_b64_tr_b16) has lanes
// 0..31 fetch 32 bytes (16 rows) from each of eight k-rows, 0..3 and 8..11 of the fragment, lanes 32..63 those 16
// further; the chunks are permuted so that the eight use the eight parts of the 256-byte bank window.  Lanes form groups
// of 16; group g covers k 8 g .. + 8; inside a group lane j supplies the 8 bytes at k-row j/4, rows 4 (j%4) .. +4, and
// receives k-rows 0..3 of row j.
template <int R, int NW, int BK = 64, bool ONCE = false> struct RowsTrans {
    static constexpr int kLoads = R * BK / (512 * NW);
    static constexpr int kChunks = R / 8;          // 16-byte chunks of a k-row
    static constexpr int kRun = BK / NW < 8 ? BK / NW : 8;   // k-rows that a wave loads at a time, all with k and 8 alike
    static constexpr int kGroup = R * kRun / 512;  // ... in so many loads
    static constexpr int kWindow = 16;             // chunks that trade places
    // R = 256: a load is two k-rows, those of a wave 4 apart, so that the permutation is the same in all of its loads
    static constexpr int kPeriod = R == 384 ? 3 : 1;   // loads until (permutation, chunk) repeat
    static constexpr int kPeriodRows = kPeriod * 64 / kChunks;    // k-rows they cover
    static_assert(kLoads * 512 * NW == R * BK && kLoads % kGroup == 0 && kGroup % kPeriod == 0 && kRun * NW % 16 == 0,
                  "the rows divide over the waves");
    static_assert(kChunks % kWindow == 0, "the permutation stays inside a window");
    static __device__ __forceinline__ int perm(int kr) {
        return ((kr & 3) | (kr >> 1 & 4)) << 1;
    }
    static __device__ __forceinline__ int first_row(int wave, int i) {   // R = 256
        return (wave & 1) * 2 + (wave >> 1) * 8 + (i & 1) * 4 + (i >> 1) * (4 * NW);
    }
    i32x4 rsrc;
    uint32_t voff[kPeriod];
    uint32_t k_step;
    uint32_t frag_base, frag_perm;
    int frag_pair;
    __device__ __forceinline__ void init(const bf16 *base, int ld, int row0, int rowlim, int klim,
                                         int lane, int wave) {
        rsrc = make_rsrc(base, (uint32_t)klim * (uint32_t)ld * 2u);
        k_step = (uint32_t)ld * 2u;
#pragma unroll
        for (int i = 0; i < kPeriod; ++i) {
            const int at = (R == 256 ? 0 : wave * kGroup + i) * 64 + lane;   // chunk of the stage the lane fills
            const int kr = at / kChunks + (R == 256 ? first_row(wave, 0) : 0);
            const int c = at % kChunks ^ perm(kr);
            const int row = row0 + (c << 3);
            voff[i] = row < rowlim ? ((uint32_t)kr * (uint32_t)ld + (uint32_t)row) * 2u : kOobOffset;
        }
    }
    // frag_row: a multiple of 32, the same for the whole wave
    __device__ __forceinline__ void init_frag16(int lane, int frag_row) {
        const int g = lane >> 4, j = lane & 15;
        const int kr = g * 8 + (j >> 2);
        frag_base = (uint32_t)(kr * (R * 2) + ((j & 3) << 3));
        frag_perm = (uint32_t)perm(kr) << 4;
        frag_pair = frag_row >> 5;
    }
    // Call it in each half step: the fragments' addresses differ by more than a constant, and the compiler would keep one
    // per fragment in registers over the k loop instead of an instruction per read.
    __device__ __forceinline__ void reload_frag() { asm volatile("" : "+v"(frag_perm)); }
    __device__ __forceinline__ void issue_one(uint32_t st, int k0, int wave, int i) const {
        if (R == 256) {
            const int row = first_row(wave, i) - first_row(wave, 0);
            dma16<ONCE>(rsrc, voff[0], (uint32_t)(k0 + row) * k_step, st + (uint32_t)(first_row(wave, i) * (R * 2)));
            return;
        }
        // load i: k-rows kRun NW (i / kGroup) + kRun wave + ..
        const int in = i % kGroup, at = i / kGroup * kRun * NW;
        dma16<ONCE>(rsrc, voff[in % kPeriod], (uint32_t)(k0 + at + in / kPeriod * kPeriodRows) * k_step,
              st + (uint32_t)(at * (R * 2) + (wave * kGroup + in) * 1024));
    }
    __device__ __forceinline__ bf16x8 frag16(const char *st, int x, int ks) const {
        typedef __attribute__((address_space(3))) s16x4 *lds_s16x4_ptr;
        constexpr uint32_t kPairs = kWindow / 4;            // 32 columns, 64 bytes, each
        const uint32_t c = (uint32_t)(frag_pair + x / 2);
        const char *p0 = st + ((frag_perm ^ (c % kPairs << 6 | (uint32_t)(x & 1) << 5)) +
                               (frag_base + c / kPairs * (kPairs * 64))) + ks * (32 * R * 2);
        const s16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4_ptr)(p0));
        const s16x4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4_ptr)(p0 + 4 * R * 2));
        return __builtin_bit_cast(bf16x8, __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7));
    }
};

// bytes per row of the epilogue's turn-around buffer of a wave with 32 IP columns (96 columns: 13 chunks, an
// odd number, so that 16 consecutive rows begin in 16 different places of the 256-byte bank window)
constexpr int rows_turn_pitch(int IP) { return IP == 1 ? 64 : IP == 2 ? 128 : 208; }

// wait until at most N of this wave's direct loads are still in flight
template <int N> __device__ __forceinline__ void rows_wait_vmcnt() {
    static_assert(N >= 0 && N < 64, "the counter has six bits");
    asm volatile("s_waitcnt vmcnt(%0)" : : "n"(N) : "memory");
}

}  // namespace sw
