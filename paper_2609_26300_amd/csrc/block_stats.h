// block_stats.h -- the block summary routine shared by the prefill, the append and the fused decode
// step (private to libcompkv): a workgroup's and a wave's, which add in the same order, so a summary does not
// depend on which of them computed it (Section 4.2: an appended block's summary equals a rebuild).
#pragma once

#include "internal.h"

namespace compkv {

// A block's summary in LDS: all that a workgroup needs that forms none itself.
template <int D>
struct BlockMeansLds {
    alignas(16) float km[D];
    alignas(16) float vm[D];
    float dv[D];
};

template <int D>
struct BlockStatsLds : BlockMeansLds<D> {
    // partial sums of each row group of each wave (4 waves of 64 / (d/8) groups): key, value; later the
    // squared deviations in the key's place
    alignas(16) float part[4][64 / (D / 8)][2][D];
};

// Summary of one block of nb >= 1 rows (row j at Kb + j*D; row new_j, if >= 0, is read from k_new /
// v_new instead of the cache): mean key, mean value and the r grouped population variances of
// Section 4.1 (Appendix A.4 groups). Called by all four waves of the workgroup with uniform arguments.
//
// A row of d bf16 is d/8 lanes x 16 bytes; a wave covers 64/(d/8) rows per load step and the workgroup
// four times that. Wave w takes rows 16s + 4w + (lane / 16) (for d = 128) of each step s, up to four
// steps per batch with every load of a batch issued before use. Per-lane sums over the rows, then the
// four waves' sums of each row group ((w0 + w1) + (w2 + w3)), then the row groups pairwise
// ((g0 + g1) + (g2 + g3), ...): the order in which one wave that plays all four (build_stats_wave_kernel) needs
// a single butterfly over its lanes instead of one per wave played. Two passes (mean, then
// squared deviations from the mean) keep the variance stable; a block of at most one batch per wave
// (64 rows for d = 128) is still in registers for the second pass. On return the results are written
// to km_out / vm_out / dv_out and their copies in L.km / L.vm / L.dv are visible to the workgroup.
//
// The first batch's loads are separate (BlockRows / load_block_rows) so that a caller can request the
// next block's rows before computing the current one.
constexpr int kStatsSteps = 4;  // load steps per batch held in registers

struct BlockSrc {
    const uint16_t* Kb;
    const uint16_t* Vb;
    const uint16_t* k_new;
    const uint16_t* v_new;
    int nb, new_j;
};

struct BlockRows {
    uint4 kw[kStatsSteps], vw[kStatsSteps];
};

template <int D>
__device__ __forceinline__ int stats_row(int st) {
    constexpr int LPR = D / 8, RPW = 64 / LPR, RPG = 4 * RPW;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    return st * RPG + wave * RPW + lane / LPR;
}

template <int D>
__device__ __forceinline__ const uint16_t* stats_krow(const BlockSrc& b, int j) {
    return (j == b.new_j) ? b.k_new : b.Kb + (size_t)j * D;
}
template <int D>
__device__ __forceinline__ const uint16_t* stats_vrow(const BlockSrc& b, int j) {
    return (j == b.new_j) ? b.v_new : b.Vb + (size_t)j * D;
}

// rows of the batch starting at step s0 (branch-free: a row past the block reloads row 0, unused)
template <int D>
__device__ __forceinline__ void load_block_rows(const BlockSrc& b, int s0, BlockRows& R, bool values = true) {
    const int li = (threadIdx.x & 63) % (D / 8);
#pragma unroll
    for (int st = 0; st < kStatsSteps; ++st) {
        const int j = stats_row<D>(s0 + st);
        const int jj = j < b.nb ? j : 0;
        R.kw[st] = *reinterpret_cast<const uint4*>(stats_krow<D>(b, jj) + li * 8);
        if (values) R.vw[st] = *reinterpret_cast<const uint4*>(stats_vrow<D>(b, jj) + li * 8);
    }
}

__device__ __forceinline__ void store_group_sums(float* p, const float (&x)[8]) {
    reinterpret_cast<float4*>(p)[0] = make_float4(x[0], x[1], x[2], x[3]);
    reinterpret_cast<float4*>(p)[1] = make_float4(x[4], x[5], x[6], x[7]);
}

// total of coordinate c over the waves, then over the row groups (the order stated above)
template <int D>
__device__ __forceinline__ float group_sum(const BlockStatsLds<D>& L, int which, int c) {
    constexpr int RPW = 64 / (D / 8);
    float t[RPW];
#pragma unroll
    for (int g = 0; g < RPW; ++g)
        t[g] = (L.part[0][g][which][c] + L.part[1][g][which][c]) + (L.part[2][g][which][c] + L.part[3][g][which][c]);
#pragma unroll
    for (int h = 1; h < RPW; h <<= 1)
#pragma unroll
        for (int g = 0; g < RPW; g += 2 * h) t[g] = t[g] + t[g + h];
    return t[0];
}

// The summary from the rows of the first batch (already requested into R) and the rest of the block.
// In a workgroup larger than four waves only waves 0-3 work (`active`); every thread reaches the
// barriers.
template <int D>
__device__ void block_stats_from(const BlockSrc& b, BlockRows& R, int r, int layout, float* __restrict__ km_out,
                                 float* __restrict__ dv_out, float* __restrict__ vm_out, BlockStatsLds<D>& L,
                                 bool active = true) {
    constexpr int LPR = D / 8;     // lanes per row
    constexpr int RPW = 64 / LPR;  // rows per wave step
    constexpr int RPG = 4 * RPW;   // rows per workgroup step
    constexpr int NS = kStatsSteps;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int ro = lane / LPR, li = lane % LPR;
    const int nb = b.nb;
    const int nsteps = (nb + RPG - 1) / RPG;

    float sk[8] = {0, 0, 0, 0, 0, 0, 0, 0}, sv[8] = {0, 0, 0, 0, 0, 0, 0, 0};
    for (int s0 = 0; active && s0 < nsteps; s0 += NS) {
        if (s0 > 0) load_block_rows<D>(b, s0, R);
#pragma unroll
        for (int st = 0; st < NS; ++st) {
            const bool ok = stats_row<D>(s0 + st) < nb;
            float kf[8], vf[8];
            unpack_bf16x8(R.kw[st], kf);
            unpack_bf16x8(R.vw[st], vf);
#pragma unroll
            for (int e = 0; e < 8; ++e) {
                sk[e] += ok ? kf[e] : 0.0f;
                sv[e] += ok ? vf[e] : 0.0f;
            }
        }
    }
    if (active) {
        store_group_sums(&L.part[wave][ro][0][li * 8], sk);
        store_group_sums(&L.part[wave][ro][1][li * 8], sv);
    }
    __syncthreads();
    const float fn = (float)nb;
    for (int i = tid; i < 2 * D; i += kThreads) {  // (threads below 256: the key's means, then the value's)
        const int which = i / D, c = i - which * D;
        const float mean = group_sum<D>(L, which, c) / fn;
        (which ? L.vm : L.km)[c] = mean;
        (which ? vm_out : km_out)[c] = mean;
    }
    __syncthreads();
    float mk[8], m2[8];
#pragma unroll
    for (int e = 0; e < 8; ++e) {
        mk[e] = L.km[li * 8 + e];
        m2[e] = 0.0f;
    }
    for (int s0 = 0; active && s0 < nsteps; s0 += NS) {
        if (nsteps > NS) load_block_rows<D>(b, s0, R, false);  // larger blocks: reload (L1/L2 hits)
#pragma unroll
        for (int st = 0; st < NS; ++st) {
            const bool ok = stats_row<D>(s0 + st) < nb;
            float kf[8];
            unpack_bf16x8(R.kw[st], kf);
#pragma unroll
            for (int e = 0; e < 8; ++e) {
                const float dev = kf[e] - mk[e];
                m2[e] += ok ? __fmul_rn(dev, dev) : 0.0f;  // (no fused multiply-add: same bits everywhere)
            }
        }
    }
    if (active) store_group_sums(&L.part[wave][ro][0][li * 8], m2);
    __syncthreads();
    auto m2_of = [&](int i) { return group_sum<D>(L, 0, i); };
    if (r == D) {
        for (int t = tid; t < D; t += kThreads) {
            const float dv = m2_of(t) / fn;
            L.dv[t] = dv;
            dv_out[t] = dv;
        }
    } else if (wave == 0) {
        // group t = a run of (d/2)/r consecutive frequency pairs (Appendix A.4); lane f holds pair f
        const bool in = lane < D / 2;
        const int f = in ? lane : 0;
        const int ia = layout == 0 ? f : 2 * f, ib = layout == 0 ? f + D / 2 : 2 * f + 1;
        float e = in ? m2_of(ia) + m2_of(ib) : 0.0f;
        const int w = (D / 2) / r;
        for (int off = 1; off < w; off <<= 1) e = xor_add(e, off);
        if (in && lane % w == 0) {
            const float dv = e / (fn * (float)(D / r));
            L.dv[lane / w] = dv;
            dv_out[lane / w] = dv;
        }
    }
    __syncthreads();
}

// The same summary computed by ONE wave (no barrier, no LDS) for blocks of at most NS workgroup load
// steps (NS * 4 * 64/(d/8) rows). The wave plays the four waves of the workgroup routine (virtual wave v
// takes the rows the real wave v takes there) and adds in exactly the same order: per lane over the steps,
// the four waves' sums, the butterflies over the row groups, the pair sums and the group butterflies over
// lanes = pairs. So its results are bit-identical to block_stats_from's, which the append and the fused step
// keep using, also where rows hold infinities or NaNs (which NaN aside).
template <int D>
constexpr int wave_stats_max_rows(int steps) {
    return steps * 4 * (64 / (D / 8));
}

// The rows of one of the block's two arrays held by a wave: [step][virtual wave]
template <int NS>
struct WaveRows {
    uint4 w[NS][4];
};

// Requests steps [s0, s0 + NS) of a block of nb rows at p (branch-free: rows past the block reload row 0)
template <int D, int NS>
__device__ __forceinline__ void load_wave_rows(const uint16_t* p, int nb, int s0, WaveRows<NS>& R) {
    constexpr int LPR = D / 8, RPW = 64 / LPR, RPG = 4 * RPW;
    const int lane = threadIdx.x & 63, ro = lane / LPR, li = lane % LPR;
#pragma unroll
    for (int st = 0; st < NS; ++st)
#pragma unroll
        for (int v = 0; v < 4; ++v) {
            const int j = (s0 + st) * RPG + v * RPW + ro;
            // (a wave-uniform base and a 32-bit byte offset)
            const unsigned off = (unsigned)(j < nb ? j : 0) * (2 * D) + li * 16;
            R.w[st][v] = load_once(reinterpret_cast<const char*>(p) + off);
        }
}

// x / n for a wave-uniform count n: for a power of two the product with its exact reciprocal, the same bits
__device__ __forceinline__ void divide8(float (&x)[8], int n) {
    if ((n & (n - 1)) == 0) {
        const float inv = 1.0f / (float)n;
#pragma unroll
        for (int e = 0; e < 8; ++e) x[e] *= inv;
    } else {
        const float fn = (float)n;
#pragma unroll
        for (int e = 0; e < 8; ++e) x[e] /= fn;
    }
}

// Keeps the compiler from carrying the rows' unpacked values (four times the registers) past this point
template <int NS>
__device__ __forceinline__ void pin_rows(WaveRows<NS>& R) {
#pragma unroll
    for (int st = 0; st < NS; ++st)
#pragma unroll
        for (int v = 0; v < 4; ++v)
            __asm__ volatile("" : "+v"(R.w[st][v].x), "+v"(R.w[st][v].y), "+v"(R.w[st][v].z), "+v"(R.w[st][v].w));
}

// Adds the rows to the lane's per-virtual-wave sums s[v][8] (kDev: the squared deviations from mk instead).
// A row past the block (a reload of row 0) enters with factor 0: fma(1, x, s) rounds like s + x, so the mask
// costs one instruction per row instead of one per value. Where row 0's value (or its square) is not finite,
// the product is NaN and so is the sum: the caller then takes wave_block_alone.
template <int D, int NS, bool kDev>
__device__ __forceinline__ void add_wave_rows(const WaveRows<NS>& R, int nb, int s0, const float (&mk)[8], float (&s)[4][8]) {
    constexpr int LPR = D / 8, RPW = 64 / LPR, RPG = 4 * RPW;
    const int ro = (threadIdx.x & 63) / LPR;
#pragma unroll
    for (int st = 0; st < NS; ++st)
#pragma unroll
        for (int v = 0; v < 4; ++v) {
            const float in = (s0 + st) * RPG + v * RPW + ro < nb ? 1.0f : 0.0f;
            float f[8];
            unpack_bf16x8(R.w[st][v], f);
#pragma unroll
            for (int e = 0; e < 8; ++e) {
                float x = f[e];
                if constexpr (kDev) {
                    const float dev = f[e] - mk[e];
                    x = __fmul_rn(dev, dev);
                }
                s[v][e] = __builtin_fmaf(in, x, s[v][e]);
            }
        }
}

template <int D>
__device__ __forceinline__ void add_row_groups(float (&t)[8]) {
#pragma unroll
    for (int off = D / 8; off < 64; off <<= 1)
#pragma unroll
        for (int e = 0; e < 8; ++e) t[e] = xor_add(t[e], off);
}

// ((w0 + w1) + (w2 + w3)), then over the row groups: every lane of a column holds the column's total
template <int D>
__device__ __forceinline__ void total_wave_rows(const float (&s)[4][8], float (&t)[8]) {
#pragma unroll
    for (int e = 0; e < 8; ++e) t[e] = (s[0][e] + s[1][e]) + (s[2][e] + s[3][e]);
    add_row_groups<D>(t);
}

__device__ __forceinline__ void zero_sums(float (&s)[4][8]) {
#pragma unroll
    for (int v = 0; v < 4; ++v)
#pragma unroll
        for (int e = 0; e < 8; ++e) s[v][e] = 0.0f;
}

// Whether one of the wave's sums is not finite (or their total overflows, which is harmless: see the caller)
__device__ __forceinline__ bool any_not_finite(const float (&t)[8]) {
    const float x = ((t[0] + t[1]) + (t[2] + t[3])) + ((t[4] + t[5]) + (t[6] + t[7]));
    return __any(!(fabsf(x) < INFINITY));
}

// The grouped variances from the coordinates' sums of squared deviations m2 (lane li: 8 li .. 8 li + 7)
template <int D>
__device__ __forceinline__ void store_wave_variances(float (&m2)[8], int nb, int r, int layout,
                                                     float* __restrict__ dv_out) {
    constexpr int LPR = D / 8;
    const int lane = threadIdx.x & 63, ro = lane / LPR, li = lane % LPR;
    const float fn = (float)nb;
    if (r == D) {
        divide8(m2, nb);
        if (ro == 0) {
#pragma unroll
            for (int e = 0; e < 8; ++e) dv_out[li * 8 + e] = m2[e];
        }
        return;
    }
    // lane f = pair f: its two coordinates' totals, fetched from the lanes that hold them
    auto coord = [&](int c) {  // every lane active; the value of coordinate c (lane c / 8, element c % 8)
        float x = 0.0f;
#pragma unroll
        for (int e = 0; e < 8; ++e) {
            const float y = __shfl(m2[e], c / 8);
            x = (c % 8 == e) ? y : x;
        }
        return x;
    };
    const bool in = lane < D / 2;
    const int f = in ? lane : 0;
    const int ia = layout == 0 ? f : 2 * f, ib = layout == 0 ? f + D / 2 : 2 * f + 1;
    const float xa = coord(ia), xb = coord(ib);
    float e2 = in ? xa + xb : 0.0f;
    const int w = (D / 2) / r;
    for (int off = 1; off < w; off <<= 1) e2 = xor_add(e2, off);
    if (in && lane % w == 0) dv_out[lane / w] = e2 / (fn * (float)(D / r));
}

// The summary of one block by one wave from the block's own rows alone, read again from memory, in the same
// order of sums: for the rare wave that met a block whose sums are not finite.
template <int D>
__device__ void wave_block_alone(const uint16_t* Kb, const uint16_t* Vb, int nb, int r, int layout,
                                    float* __restrict__ km_out, float* __restrict__ dv_out, float* __restrict__ vm_out) {
#pragma clang fp contract(off)  // (the rounded square is added, as in the workgroup routine: the same bits)
    constexpr int LPR = D / 8, RPW = 64 / LPR, RPG = 4 * RPW;
    const int lane = threadIdx.x & 63, ro = lane / LPR, li = lane % LPR;
    float mean[8] = {0, 0, 0, 0, 0, 0, 0, 0}, t[8] = {0, 0, 0, 0, 0, 0, 0, 0};
#pragma unroll 1
    for (int pass = 0; pass < 3; ++pass) {  // values, keys, the keys' squared deviations
        const uint16_t* p = pass == 0 ? Vb : Kb;
        float pair[8] = {0, 0, 0, 0, 0, 0, 0, 0};
#pragma unroll 1
        for (int v = 0; v < 4; ++v) {  // (w0 + w1) + (w2 + w3)
            float s[8] = {0, 0, 0, 0, 0, 0, 0, 0};
#pragma unroll 1
            for (int j = v * RPW + ro; j < nb; j += RPG) {
                float f[8];
                unpack_bf16x8(*reinterpret_cast<const uint4*>(p + (size_t)j * D + li * 8), f);
#pragma unroll
                for (int e = 0; e < 8; ++e) {
                    const float dev = f[e] - mean[e];
                    s[e] += pass == 2 ? __fmul_rn(dev, dev) : f[e];
                }
            }
#pragma unroll
            for (int e = 0; e < 8; ++e) {
                t[e] = v == 1 ? pair[e] + s[e] : v == 3 ? t[e] + (pair[e] + s[e]) : t[e];
                pair[e] = s[e];
            }
        }
        add_row_groups<D>(t);
        if (pass == 2) break;
        divide8(t, nb);
        float* out = pass == 0 ? vm_out : km_out;
#pragma unroll
        for (int e = 0; e < 8; ++e) {
            mean[e] = t[e];
            if (ro == 0) out[li * 8 + e] = t[e];
        }
    }
    store_wave_variances<D>(t, nb, r, layout, dv_out);
}

template <int D>
__device__ void wg_block_stats(const uint16_t* __restrict__ Kb, const uint16_t* __restrict__ Vb, int nb,
                               const uint16_t* __restrict__ k_new, const uint16_t* __restrict__ v_new, int new_j,
                               int r, int layout, float* __restrict__ km_out, float* __restrict__ dv_out,
                               float* __restrict__ vm_out, BlockStatsLds<D>& L) {
    const BlockSrc b{Kb, Vb, k_new, v_new, nb, new_j};
    BlockRows R;
    load_block_rows<D>(b, 0, R);
    block_stats_from<D>(b, R, r, layout, km_out, dv_out, vm_out, L);
}

}  // namespace compkv
