// Position assignment, dispatch gather, combine scatter and its backward.
// All of these stream rows through HBM once; they are laid out so that a wave
// moves whole 16-byte chunks of a row with every lane busy.
#include "common.h"
#include "router_wgrad.h"

namespace sw {

// 16-byte chunk of a row
struct __attribute__((aligned(16))) Chunk16 {
    uint32_t w[4];
};

template <typename XT> struct Vec;
template <> struct Vec<bf16> { static constexpr int N = 8; };
template <> struct Vec<float> { static constexpr int N = 4; };

template <typename XT> __device__ __forceinline__ void unpack(const Chunk16 &c, float *v);
template <> __device__ __forceinline__ void unpack<float>(const Chunk16 &c, float *v) {
#pragma unroll
    for (int i = 0; i < 4; ++i) v[i] = __uint_as_float(c.w[i]);
}
template <> __device__ __forceinline__ void unpack<bf16>(const Chunk16 &c, float *v) {
#pragma unroll
    for (int i = 0; i < 4; ++i) {   // bf16 -> fp32 is a 16-bit shift
        v[2 * i] = __uint_as_float(c.w[i] << 16);
        v[2 * i + 1] = __uint_as_float(c.w[i] & 0xffff0000u);
    }
}
template <typename XT> __device__ __forceinline__ Chunk16 pack(const float *v);
template <> __device__ __forceinline__ Chunk16 pack<float>(const float *v) {
    Chunk16 c;
#pragma unroll
    for (int i = 0; i < 4; ++i) c.w[i] = __float_as_uint(v[i]);
    return c;
}
template <> __device__ __forceinline__ Chunk16 pack<bf16>(const float *v) {
    Chunk16 c;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        typedef bf16 bf16x2 __attribute__((ext_vector_type(2)));
        bf16x2 pr;
        pr[0] = (bf16)v[2 * i];       // round to nearest even
        pr[1] = (bf16)v[2 * i + 1];
        c.w[i] = __builtin_bit_cast(uint32_t, pr);
    }
    return c;
}

// Passes with one wave per token: blocks of four tokens, 2^23 of them (2^31 threads) in the grid's first
// dimension, more than 2^25 tokens in the second.
constexpr int kRowBlocks = 1 << 23;
static dim3 row_grid(int64_t T) {
    const int64_t blocks = ceil_div(T, 256 / kWave);
    return dim3((unsigned)(blocks < kRowBlocks ? blocks : kRowBlocks), (unsigned)ceil_div(blocks, kRowBlocks));
}
__device__ __forceinline__ uint32_t wave_token() {
    return (blockIdx.y * kRowBlocks + blockIdx.x) * (256 / kWave) + threadIdx.x / kWave;
}

// -----------------------------------------------------------------------------
// Assign, 16 tokens per block (a token block of the routing tables is shared by several):
// position_in_expert[t] = block_off[block(t)][e_t] + local_rank[t] (rank inside the token's
// routing group); dropped mask (position >= Cg); slot of each kept token,
// e * C + grp_off[g][e] + position, the slot -> token table and the gate of each slot's token;
// then (COPY) the dispatch gather Xd[slot] = x[t] of the block's kept tokens.
// INLINE: the prefix sums of the block histograms are taken here instead of being read from the
// scan kernel's tables, and one more block does what is left of that kernel: counts, kept, the
// loss.  With few token blocks and experts that costs less than a launch (T = 2048: 10 us; scan, positions
// and gather as three launches took 27); see scan_inline for where it does not.  16 tokens per block: with 64, a gather of 16384 rows of
// 8 KB took 97 us on its 256 blocks, with 16 it takes 53, as the row-per-wave pass it replaces.
// -----------------------------------------------------------------------------
struct AssignArgs {
    const int32_t *idx, *local_rank, *block_counts, *block_off;
    const float *block_psum, *gate;
    int32_t *grp_off, *counts, *kept, *counts_g;
    int32_t *hit;               // (null: not counted)
    int32_t *pos_out, *counts_out;
    uint8_t *dropped_out;
    int32_t *slot_token;
    float *slot_gate;
    uint32_t *slot_off;          // only with dispatch inside the GEMMs
    uint32_t row_bytes;
    int32_t *tok_slot;
    const double *loss_part;
    int loss_parts;
    double loss_scale;           // alpha E / n
    float *aux_out;
    int tb, nbg, nb, n, Tg, E, C, Cg;
    const Chunk16 *x;            // COPY
    Chunk16 *Xd;
    Chunk16 *y_zero;             // rows of tokens without a slot become +0, or null
    int cpr;                     // 16-byte chunks per row
};

// sums over rows [lo, hi) of a [..][E] table, columns e0 .. e0 + 255, into out[] (LDS); whole block.
// The threads that are not needed side by side split the rows; W columns per thread.
template <typename V, int W>
__device__ __forceinline__ void column_sums_w(const V *__restrict__ table, int lo, int hi, int E, int e0,
                                              V *part /* [256 W] */, V *out) {
    int ew = 256 / W;
    while (ew > 1 && ew / 2 * W >= E - e0) ew >>= 1;
    const int P = 256 / ew < 16 ? 256 / ew : 16;   // (the parts are added up one after the other)
    const int col = threadIdx.x % ew, p = threadIdx.x / ew;
    const int per = (hi - lo + P - 1) / P;
    const int a = lo + p * per, z = a + per < hi ? a + per : hi;
    V s[W];
#pragma unroll
    for (int m = 0; m < W; ++m) s[m] = 0;
    if (p < P && e0 + col * W < E)
#pragma unroll 8
        for (int b = a; b < z; ++b) {
            V v[W];
            __builtin_memcpy(v, __builtin_assume_aligned(table + (size_t)b * E + e0 + col * W, W * 4), W * 4);
#pragma unroll
            for (int m = 0; m < W; ++m) s[m] += v[m];
        }
#pragma unroll
    for (int m = 0; m < W; ++m) part[threadIdx.x * W + m] = s[m];
    __syncthreads();
    if ((int)threadIdx.x < ew * W) {
        V t = part[threadIdx.x];
        for (int q = 1; q < P; ++q) t += part[q * ew * W + threadIdx.x];
        out[threadIdx.x] = t;
    }
    __syncthreads();
}
template <typename V>
__device__ __forceinline__ void column_sums(const V *__restrict__ table, int lo, int hi, int E, int e0, V *part,
                                            V *out) {
    if ((E & 3) == 0) column_sums_w<V, 4>(table, lo, hi, E, e0, part, out);
    else column_sums_w<V, 1>(table, lo, hi, E, e0, part, out);
}

constexpr int kAssignTok = 16;   // tokens per block

template <bool INLINE, bool COPY>
__global__ __launch_bounds__(256) void assign_kernel(AssignArgs a) {
    __shared__ int32_t slot_s[kAssignTok];
    __shared__ int32_t part[INLINE ? 1024 : kAssignTok], sums[INLINE ? 256 : 1];
    __shared__ float fpart[INLINE ? 1024 : 1], fsums[INLINE ? 256 : 1];
    __shared__ double red[INLINE ? 256 : 1];
    __shared__ int n_dropped;
    extern __shared__ int32_t dyn[];   // INLINE: off[E], goff[E] of the block's group
    const int tid = threadIdx.x;
    const int per_b = a.tb / kAssignTok, b = blockIdx.x / per_b;
    const int E = a.E;
    if (INLINE && b == a.nb) {   // the extra block: totals over all token blocks
        double loss = 0.0;
        int hit = 0;
        for (int e0 = 0; e0 < E; e0 += 256) {
            int total = 0, kept = 0;
            for (int g = 0; g < a.n; ++g) {
                column_sums<int32_t>(a.block_counts, g * a.nbg, (g + 1) * a.nbg, E, e0, part, sums);
                column_sums<float>(a.block_psum, g * a.nbg, (g + 1) * a.nbg, E, e0, fpart, fsums);
                if (e0 + tid < E) {
                    const int c = sums[tid];
                    a.counts_g[(size_t)g * E + e0 + tid] = c;
                    total += c;
                    kept += c < a.Cg ? c : a.Cg;
                    loss += ((double)c / (double)a.Tg) * ((double)fsums[tid] / (double)a.Tg);   // Eqs. 4-6
                }
                __syncthreads();
            }
            if (e0 + tid < E) {
                a.counts[e0 + tid] = total;
                a.counts_out[e0 + tid] = total;
                a.kept[e0 + tid] = kept;
            }
            if (a.hit) hit += __syncthreads_count(kept > 0);
        }
        if (a.hit && tid == 0) *a.hit = hit;
        red[tid] = loss;
        __syncthreads();
        for (int s = 128; s >= 1; s >>= 1) {
            if (tid < s) red[tid] += red[tid + s];
            __syncthreads();
        }
        if (tid == 0) a.aux_out[0] = (float)(a.loss_scale * red[0]);
        return;
    }
    const int g = b / a.nbg;
    int t0, tend;
    block_token_range(b, a.nbg, a.Tg, a.tb, t0, tend);
    t0 += (blockIdx.x - b * per_b) * kAssignTok;   // this block's share
    tend = t0 + kAssignTok < tend ? t0 + kAssignTok : tend;
    if (t0 >= tend && blockIdx.x != 0) return;
    if (tid == 0) n_dropped = 0;
    if (INLINE) {
        for (int e0 = 0; e0 < E; e0 += 256) {
            int goff = 0;   // slots of the earlier groups
            for (int q = 0; q < g; ++q) {
                column_sums<int32_t>(a.block_counts, q * a.nbg, (q + 1) * a.nbg, E, e0, part, sums);
                if (e0 + tid < E) goff += sums[tid] < a.Cg ? sums[tid] : a.Cg;
                __syncthreads();
            }
            column_sums<int32_t>(a.block_counts, g * a.nbg, b, E, e0, part, sums);
            if (e0 + tid < E) {
                dyn[e0 + tid] = sums[tid];
                dyn[E + e0 + tid] = goff;
                if (t0 == g * a.Tg) a.grp_off[(size_t)g * E + e0 + tid] = goff;
            }
            __syncthreads();
        }
    } else {
        if (blockIdx.x == 0 && tid == 0) {   // Eqs. 4-6 from the scan's parts, in order
            double sum = 0.0;
            for (int i = 0; i < a.loss_parts; ++i) sum += a.loss_part[i];
            a.aux_out[0] = (float)(a.loss_scale * sum);
        }
        if (a.hit && blockIdx.x == 0) {
            int hit = 0;
            for (int e0 = 0; e0 < E; e0 += 256) hit += __syncthreads_count(e0 + tid < E && a.kept[e0 + tid] > 0);
            if (tid == 0) *a.hit = hit;
        }
        __syncthreads();
    }
    if (tid < kAssignTok) {
        const int t = t0 + tid;
        int slot_or_none = -1;
        if (t < tend) {
            const int e = a.idx[t];
            const int p = (INLINE ? dyn[e] : a.block_off[(size_t)b * E + e]) + a.local_rank[t];
            const uint8_t dr = p >= a.Cg;
            a.pos_out[t] = p;
            a.dropped_out[t] = dr;
            if (!dr) {
                const int slot = e * a.C + (INLINE ? dyn[E + e] : a.grp_off[(size_t)g * E + e]) + p;
                slot_or_none = slot;
                a.slot_token[slot] = t;
                a.slot_gate[slot] = a.gate[t];
                if (a.slot_off) a.slot_off[slot] = (uint32_t)t * a.row_bytes;
            }
            a.tok_slot[t] = slot_or_none;
        }
        slot_s[tid] = slot_or_none;
        if (a.y_zero && t < tend && slot_or_none < 0) part[atomicAdd(&n_dropped, 1)] = t;   // any order
    }
    if (!COPY && !a.y_zero) return;
    __syncthreads();
    if (COPY) {
        const int total = (tend - t0) * a.cpr;
#pragma unroll 4
        for (int i = tid; i < total; i += 256) {
            const int tl = i / a.cpr, c = i - tl * a.cpr;
            const int slot = slot_s[tl];
            if (slot >= 0) a.Xd[(size_t)slot * a.cpr + c] = a.x[(size_t)(t0 + tl) * a.cpr + c];
        }
    }
    if (a.y_zero) {   // the block's tokens without a slot get their rows of y: +0
        const Chunk16 zero = {{0u, 0u, 0u, 0u}};
        for (int i = tid; i < n_dropped * a.cpr; i += 256) {
            const int k = i / a.cpr;
            a.y_zero[(size_t)part[k] * a.cpr + (i - k * a.cpr)] = zero;
        }
    }
}

// -----------------------------------------------------------------------------
// Dispatch: Xd[slot_t][:] = x[t][:] for kept tokens.  One wave per token
// (its index loads are wave-uniform), one 16-byte chunk per lane and pass;
// cpr = chunks per row.
// -----------------------------------------------------------------------------
__global__ __launch_bounds__(256) void dispatch_kernel(const Chunk16 *__restrict__ x,
                                                       Chunk16 *__restrict__ Xd,
                                                       const int32_t *__restrict__ tok_slot,
                                                       int T, int cpr) {
    const int lane = threadIdx.x % kWave;
    const uint32_t t = wave_token();
    if (t >= (uint32_t)T) return;
    const int slot_or_none = tok_slot[t];
    if (slot_or_none < 0) return;
    const size_t slot = (size_t)slot_or_none;
    for (int col = lane; col < cpr; col += kWave) Xd[slot * cpr + col] = x[(size_t)t * cpr + col];
}

// -----------------------------------------------------------------------------
// Combine: y[t][:] = gate[t] * O[slot_t][:] for kept tokens, +0 for dropped.
// One wave per token.
// -----------------------------------------------------------------------------
template <typename XT>
__global__ __launch_bounds__(256) void combine_kernel(const Chunk16 *__restrict__ O,
                                                      Chunk16 *__restrict__ y,
                                                      const int32_t *__restrict__ tok_slot,
                                                      const float *__restrict__ gate,
                                                      int T, int cpr) {
    const int lane = threadIdx.x % kWave;
    const uint32_t t = wave_token();
    if (t >= (uint32_t)T) return;
    const int slot_or_none = tok_slot[t];
    if (slot_or_none < 0) {
        const Chunk16 zero = {{0u, 0u, 0u, 0u}};
        for (int col = lane; col < cpr; col += kWave) y[(size_t)t * cpr + col] = zero;
        return;
    }
    const size_t slot = (size_t)slot_or_none;
    const float g = gate[t];
    for (int col = lane; col < cpr; col += kWave) {
        const Chunk16 in = O[slot * cpr + col];
        float v[Vec<XT>::N];
        unpack<XT>(in, v);
#pragma unroll
        for (int i = 0; i < Vec<XT>::N; ++i) v[i] *= g;
        y[(size_t)t * cpr + col] = pack<XT>(v);
    }
}

// -----------------------------------------------------------------------------
// Combine backward: for kept tokens dO[slot_t][:] = gate[t] * dy[t][:] and
// dgate[t] = <dy[t], O[slot_t]>; dropped tokens get dgate = 0.  One wave per token.
// -----------------------------------------------------------------------------
// The lane's share (up to 256 experts) of the token's s = sum_i p[i] dp[i] for router_wgrad_block, without the gate's gradient,
// which enters times p_me.
__device__ __forceinline__ float lane_row_sum(const RouterWgradArgs &r, uint32_t t, int lane, float &p_me) {
    const float mean_count = (float)r.Tg / (float)r.E;
    const int32_t *counts = r.counts_g + (size_t)((int)t / r.Tg) * r.E;
    float s = 0.f;
#pragma unroll
    for (int j = 0; j < 4; ++j) {
        const int e = lane + j * kWave;
        if (e < r.E) s += r.probs[(size_t)t * r.E + e] * (r.aux_scale * ((float)counts[e] - mean_count));
    }
    p_me = r.probs[(size_t)t * r.E + r.idx[t]];
    return s;
}

template <typename XT, bool SUM>
__global__ __launch_bounds__(256) void combine_bwd_kernel(
    const Chunk16 *__restrict__ dy, const Chunk16 *__restrict__ O, Chunk16 *__restrict__ dO,
    const int32_t *__restrict__ tok_slot, const float *__restrict__ gate,
    float *__restrict__ dgate, int T, int cpr, RouterWgradArgs r, float *__restrict__ rowsum) {
    const int lane = threadIdx.x % kWave;
    const uint32_t t = wave_token();
    if (t >= (uint32_t)T) return;
    float s = 0.f, p_me = 0.f;
    if (SUM) s = lane_row_sum(r, t, lane, p_me);
    const int slot_or_none = tok_slot[t];
    float dot = 0.f;
    if (slot_or_none >= 0) {
        const size_t slot = (size_t)slot_or_none;
        const float g = gate[t];
        for (int col = lane; col < cpr; col += kWave) {
            const Chunk16 a = dy[(size_t)t * cpr + col];
            const Chunk16 b = O[slot * cpr + col];
            float av[Vec<XT>::N], bv[Vec<XT>::N];
            unpack<XT>(a, av);
            unpack<XT>(b, bv);
#pragma unroll
            for (int i = 0; i < Vec<XT>::N; ++i) {
                dot = fmaf(av[i], bv[i], dot);
                av[i] *= g;
            }
            dO[slot * cpr + col] = pack<XT>(av);
        }
    } else if (!SUM) {
        if (lane == 0) dgate[t] = 0.f;
        return;
    }
#pragma unroll
    for (int m = 32; m >= 1; m >>= 1) {
        dot += __shfl_xor(dot, m, kWave);
        if (SUM) s += __shfl_xor(s, m, kWave);
    }
    if (lane == 0) {
        dgate[t] = dot;
        if (SUM) rowsum[t] = fmaf(p_me, dot, s);
    }
}

// -----------------------------------------------------------------------------
// Dispatch and combine inside the GEMMs: what is left of the two passes.
//   zero_dropped: y[t][:] = +0 for the tokens without a slot (the second GEMM's epilogue writes
//                 the rows of all others).  One wave per token.
//   gate_grad:    dgate[t] = <dy[t], o_t> for kept tokens, 0 for dropped ones, from the saved
//                 slot-major copy of the output rows Y[slot_t] = gate[t] o_t: <dy[t], Y[slot_t]> /
//                 gate[t] (a gate that underflowed to 0 gets gradient 0: its probability is 0
//                 and so is every term the gradient would enter).  One wave per token.
// -----------------------------------------------------------------------------
__global__ __launch_bounds__(256) void zero_dropped_kernel(Chunk16 *__restrict__ y,
                                                           const int32_t *__restrict__ tok_slot,
                                                           int T, int cpr) {
    const int lane = threadIdx.x % kWave;
    const uint32_t t = wave_token();
    if (t >= (uint32_t)T || tok_slot[t] >= 0) return;
    const Chunk16 zero = {{0u, 0u, 0u, 0u}};
    for (int col = lane; col < cpr; col += kWave) y[(size_t)t * cpr + col] = zero;
}

template <typename XT, bool SUM>
__global__ __launch_bounds__(256) void gate_grad_kernel(const Chunk16 *__restrict__ dy,
                                                        const Chunk16 *__restrict__ Y,
                                                        const int32_t *__restrict__ tok_slot,
                                                        const float *__restrict__ gate,
                                                        float *__restrict__ dgate, int T, int cpr,
                                                        RouterWgradArgs r, float *__restrict__ rowsum) {
    const int lane = threadIdx.x % kWave;
    const uint32_t t = wave_token();
    if (t >= (uint32_t)T) return;
    float s = 0.f, p_me = 0.f;
    if (SUM) s = lane_row_sum(r, t, lane, p_me);
    const int slot_or_none = tok_slot[t];
    float dot = 0.f;
    if (slot_or_none >= 0) {
        const size_t slot = (size_t)slot_or_none;
        for (int col = lane; col < cpr; col += kWave) {
            float av[Vec<XT>::N], bv[Vec<XT>::N];
            unpack<XT>(dy[(size_t)t * cpr + col], av);
            unpack<XT>(Y[slot * cpr + col], bv);
#pragma unroll
            for (int i = 0; i < Vec<XT>::N; ++i) dot = fmaf(av[i], bv[i], dot);
        }
    } else if (!SUM) {
        if (lane == 0) dgate[t] = 0.f;
        return;
    }
#pragma unroll
    for (int m = 32; m >= 1; m >>= 1) {
        dot += __shfl_xor(dot, m, kWave);
        if (SUM) s += __shfl_xor(s, m, kWave);
    }
    if (lane == 0) {
        const float g = gate[t], dg = slot_or_none >= 0 && g > 0.f ? dot / g : 0.f;
        dgate[t] = dg;
        if (SUM) rowsum[t] = fmaf(p_me, dg, s);
    }
}

// -----------------------------------------------------------------------------
// launchers
// -----------------------------------------------------------------------------
hipError_t launch_zero_dropped(const Workspace &w, char *ws, void *y, hipStream_t s) {
    ProfScope ps("zero_dropped", s);
    hipLaunchKernelGGL(zero_dropped_kernel, row_grid(w.T), dim3(256), 0,
                       s, (Chunk16 *)y, (const int32_t *)(ws + w.tok_slot), (int)w.T,
                       (int)(w.d * w.elt / 16));
    return hipGetLastError();
}

hipError_t launch_gate_grad(const Workspace &w, const void *dy, char *ws, const RouterWgradArgs &parts, hipStream_t s) {
    ProfScope ps("gate_grad", s);
    hipLaunchKernelGGL((parts.blocks ? gate_grad_kernel<bf16, true> : gate_grad_kernel<bf16, false>), row_grid(w.T), dim3(256),
                       0, s, (const Chunk16 *)dy, (const Chunk16 *)(ws + w.O),
                       (const int32_t *)(ws + w.tok_slot), (const float *)(ws + w.gate),
                       (float *)(ws + w.dgate), (int)w.T, (int)(w.d / 8), parts, (float *)(ws + w.local_rank));
    return hipGetLastError();
}

hipError_t launch_dispatch(const Workspace &w, int dtype, float alpha, const void *x, char *ws,
                           int32_t *position_in_expert, uint8_t *dropped, int32_t *expert_counts,
                           float *aux_loss, const float *logits, int32_t *expert_index, float *gate,
                           void *y, hipStream_t s) {
    hipError_t err;
    const int cpr = (int)(w.d * w.elt / 16);
    // the gather of the kept tokens: here, unless re-routing stages place more of them first or the
    // GEMMs read x through the slot -> token table
    const bool gather = w.C > 0 && !w.fused, copy = gather && w.ntlb_rounds == 0;
    {
        AssignArgs a{};
        a.idx = (const int32_t *)(ws + w.idx);
        a.local_rank = (const int32_t *)(ws + w.local_rank);
        a.block_counts = (const int32_t *)(ws + w.block_counts);
        a.block_psum = (const float *)(ws + w.block_psum);
        a.block_off = (const int32_t *)(ws + w.block_off);
        a.gate = (const float *)(ws + w.gate);
        a.grp_off = (int32_t *)(ws + w.grp_off);
        a.counts = (int32_t *)(ws + w.counts);
        a.kept = (int32_t *)(ws + w.kept);
        a.counts_g = (int32_t *)(ws + w.counts_g);
        a.hit = rows_count_hit(w) ? (int32_t *)(ws + w.hit) : nullptr;
        a.pos_out = position_in_expert;
        a.counts_out = expert_counts;
        a.dropped_out = dropped;
        a.slot_token = (int32_t *)(ws + w.slot_token);
        a.slot_gate = (float *)(ws + w.slot_gate);
        a.slot_off = w.fused ? (uint32_t *)(ws + w.slot_off) : nullptr;
        a.row_bytes = (uint32_t)(w.d * w.elt);
        a.tok_slot = (int32_t *)(ws + w.tok_slot);
        a.loss_part = (const double *)(ws + w.loss_part);
        a.loss_parts = route_scan_parts(w);
        a.loss_scale = (double)alpha * (double)w.E / (double)w.n;
        a.aux_out = aux_loss;
        a.tb = w.tb; a.nbg = (int)w.nbg; a.nb = (int)w.nb; a.n = (int)w.n; a.Tg = (int)w.Tg;
        a.E = (int)w.E; a.C = (int)w.C; a.Cg = (int)w.Cg;
        a.x = (const Chunk16 *)x;
        a.Xd = (Chunk16 *)(ws + w.Xd);
        a.y_zero = zero_rows_with_positions(w) ? (Chunk16 *)y : nullptr;
        a.cpr = cpr;
        ProfScope ps("assign_gather", s);
        const dim3 grid((unsigned)(w.nb * (w.tb / kAssignTok) + (w.inline_scan ? 1 : 0)));
        const size_t dyn = w.inline_scan ? 2 * sizeof(int32_t) * (size_t)w.E : 0;
        if (w.inline_scan && copy) hipLaunchKernelGGL((assign_kernel<true, true>), grid, dim3(256), dyn, s, a);
        else if (w.inline_scan) hipLaunchKernelGGL((assign_kernel<true, false>), grid, dim3(256), dyn, s, a);
        else if (copy) hipLaunchKernelGGL((assign_kernel<false, true>), grid, dim3(256), dyn, s, a);
        else hipLaunchKernelGGL((assign_kernel<false, false>), grid, dim3(256), dyn, s, a);
        if ((err = hipGetLastError()) != hipSuccess) return err;
    }
    if (w.C == 0) return hipSuccess;
    if (w.ntlb_rounds > 0 &&
        (err = launch_ntlb(w, ws, logits, expert_index, gate, position_in_expert, dropped, s)) !=
            hipSuccess)
        return err;
    if (!gather || copy) return hipSuccess;
    ProfScope ps("dispatch_gather", s);
    hipLaunchKernelGGL(dispatch_kernel, row_grid(w.T), dim3(256), 0, s,
                       (const Chunk16 *)x, (Chunk16 *)(ws + w.Xd), (const int32_t *)(ws + w.tok_slot),
                       (int)w.T, cpr);
    return hipGetLastError();
}

hipError_t launch_combine(const Workspace &w, int dtype, char *ws, void *y, hipStream_t s) {
    ProfScope ps("combine_scatter", s);
    const int vec = dtype == SW_BF16 ? 8 : 4;
    const int cpr = (int)(w.d / vec);
    const dim3 grid = row_grid(w.T);
    if (dtype == SW_BF16)
        hipLaunchKernelGGL(combine_kernel<bf16>, grid, dim3(256), 0, s,
                           (const Chunk16 *)(ws + w.O), (Chunk16 *)y,
                           (const int32_t *)(ws + w.tok_slot), (const float *)(ws + w.gate),
                           (int)w.T, cpr);
    else
        hipLaunchKernelGGL(combine_kernel<float>, grid, dim3(256), 0, s,
                           (const Chunk16 *)(ws + w.O), (Chunk16 *)y,
                           (const int32_t *)(ws + w.tok_slot), (const float *)(ws + w.gate),
                           (int)w.T, cpr);
    return hipGetLastError();
}

hipError_t launch_combine_bwd(const Workspace &w, int dtype, const void *dy, char *ws, const RouterWgradArgs &parts,
                              hipStream_t s) {
    ProfScope ps("combine_bwd", s);
    auto launch = [&](auto kern, int vec) {
        hipLaunchKernelGGL(kern, row_grid(w.T), dim3(256), 0, s, (const Chunk16 *)dy, (const Chunk16 *)(ws + w.O),
                           (Chunk16 *)(ws + w.dO), (const int32_t *)(ws + w.tok_slot), (const float *)(ws + w.gate),
                           (float *)(ws + w.dgate), (int)w.T, (int)(w.d / vec), parts, (float *)(ws + w.local_rank));
    };
    if (dtype == SW_BF16) {
        if (parts.blocks) launch(combine_bwd_kernel<bf16, true>, 8);
        else launch(combine_bwd_kernel<bf16, false>, 8);
    } else {
        if (parts.blocks) launch(combine_bwd_kernel<float, true>, 4);
        else launch(combine_bwd_kernel<float, false>, 4);
    }
    return hipGetLastError();
}

}  // namespace sw
