// select.hip -- block scoring and Top-K selection (Sections 4.1, 4.2; Appendix E.1).
//
// Launch 1, grid = units * (nchunks + 1), one-dimensional. Chunk workgroups stream the fp32 summaries
// (mean key, grouped variances) of `bpc` consecutive blocks of one unit. Eight lanes share a block: lane
// i of the eight reads float4 i, i+8, ... of the mean-key row (the eight lanes read 128 contiguous bytes
// per load) and the variance groups t = i, i+8, .... The sequence length and the query are requested
// first and the query is in LDS before any mean key is requested (a CU returns loads in request order,
// so a query requested after the other workgroups' mean keys would wait behind them); then two slots of
// 32 blocks are in flight, slot p + 2 requested once slot p is computed (block ids are clamped to the
// allocated range and masked afterwards). For each of the unit's G query heads a workgroup forms the
// block-mean logit zbar = s q.kmean, the projected variance sig2 = s^2 sum_t Q_t dvar_t and the log
// weight estimate a = log|b| + zbar + sig2/2 (the log of the numerator of Eq. compkv-mass-estimate). It
// writes zbar (block logits, reused by the decode), the chunk's per-head (max m_c of a, sum of
// exp(a - m_c)), and per block the G terms w_g = exp(a_g - m_c) sig2_g, stored contiguously so one
// vector load fetches a block's terms. The last block of each unit (the one a decode step appends to) is
// scored by one extra workgroup per unit, which writes its own partial; the chunks skip it. When every
// workgroup is resident at once these lead the grid (dispatched first, they are no longer the last to
// finish); otherwise they trail it, so that the chunks (the long pole) all start at once.
//
// Fused decode step (kStep): the extra workgroup first stores the new row and recomputes the last
// block's summary with the append's routine (bit-identical), so no chunk waits for it, and zeroes the
// unit's words for the fused selection/exact launch. On the chunked shape every workgroup also forms the
// compensation partial of its blocks (pseudo-logits log|b| + zbar, weights exp(. - max), weighted mean
// values); on the chunked-exact shape the fused launch streams the mean values instead.
//
// Launch 2 (chunked shape), grid = units: the kernel boundary makes every partial visible. One
// workgroup per unit merges the partials into each head's log normalizer lse_g and forms
// S_b = sum_g exp(m_c - lse_g) w_g (= Eq. compkv-score). Block b is ranked by the 64-bit key
// (bits of S_b) << 32 | ~b: scores are >= 0, so their IEEE bit patterns order like the values, and the
// keys are unique and order exactly like (S_b descending, b ascending), the stable Top-K of the paper.
// Up to 8192 blocks the keys stay in registers (eight per thread of 1024). One histogram of each key's
// distance below the largest score (bins of 1/16 octave on the float bits; keys farther than 255 bins
// are not counted) locates the bin that holds the (K-|F|)-th largest key; only the keys in that bin or
// above are ranked exactly, by brute force, and a bitmap of the selected and mandatory blocks is
// compacted into ascending ids. Larger inputs, or ties that leave too many keys at or above the cut's
// bin, go through a three-pass radix select on the score bits instead. Wave-level reductions and prefix
// sums use DPP lane moves. (select_core.h holds this selection, shared with the fused launches.)
//
// The chunked-exact shape replaces launch 2 and the decode's launches by one fused selection/exact
// launch in one of two forms (fused.hip): item workgroups that each select and attend, beside compensation
// workgroups that stream the mean values; or one selector per unit whose ids the unit's other
// workgroups take from a mailbox after streaming their share of the mean values. Either form merges the
// unit's partials in the launch (its last workgroup).
#include "select_core.h"

namespace compkv {
namespace {

// Per-block LDS rows of a chunk of 32 PMAX blocks: at least one wave's width, since the per-head passes
// give every lane of a wave a slot. Sizing them by the chunk (not the largest one) keeps the 64-block
// chunks of G = 8 at five workgroups per CU.
template <int PMAX>
constexpr int chunk_slots() {
    return 32 * PMAX < 64 ? 64 : 32 * PMAX;
}

template <int D, int G, int NB>
struct ChunkShared {
    float q[G][D];   // scaled query
    float Qv[G][D];  // s^2 * sum of q^2 over each group (first r entries)
    float z[G][NB];
    float v[G][NB];  // (a block's log weight is formed from z and v where it is needed)
    float m[G];
};

// Compensation state of the fused decode step.
template <int D, int G, int NB>
struct CompShared {
    float cw[G][NB];
    float cm[G], cl[G];
    alignas(16) float acc[4][G][D];
};
struct NoComp {};

template <int D, int G, bool kStep>
struct TailShared {
    // the last block's summary (km, vm, dv); the scoring call forms none, so its workgroups go without the 16 KB of
    // partial sums (19 to 26 KB a workgroup with them, 7 to 16 without: 8 waves per SIMD again instead of 6 at G = 8)
    std::conditional_t<kStep, BlockStatsLds<D>, BlockMeansLds<D>> bs;
    float q[G][D];
    float Qv[G][D];
    float z[G], v[G];
};

// A chunk workgroup and a last-block workgroup share one LDS allocation.
template <int D, int G, bool kStep, int NB>
union ChunkLds {
    struct {
        ChunkShared<D, G, NB> sh;
        std::conditional_t<kStep, CompShared<D, G, NB>, NoComp> st;
    } c;
    TailShared<D, G, kStep> t;
};

// The extra workgroup of unit u: the last block X - 1 (refreshed first when the step appends).
template <int D, int G, bool kStep>
__device__ void score_tail(const Geom& geo, const ScoreArgs& a, int u, TailShared<D, G, kStep>& ts) {
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int bseq = u / geo.hkv, h = u % geo.hkv;
    const int nc = a.nchunks;
    const uint16_t* qh = a.q + ((size_t)bseq * geo.hq + (size_t)h * G) * D;
    QueryPairs<D, G> qp;
    load_query_pairs<D, G>(qh, geo.layout, qp);  // consumed only after the block's own loads are issued
    const int n_raw = a.seq_lens[bseq];
    const int n = clamp_len(n_raw, geo.max_seq);
    const int X = (n + geo.B - 1) / geo.B;
    float* pp = a.ws_part + ((size_t)u * (nc + 1) + nc) * G * 2;
    if (a.arrive_zero) {  // for the launch that merges after this one
        if (tid == 0) a.arrive_zero[u] = 0u;
        uint32_t* mbox = a.arrive_zero + (size_t)geo.units() + (size_t)u * a.K;
        for (int k = tid; k < a.K; k += kThreads) mbox[k] = 0u;
    }
    // fused step with Mean compensation: this workgroup's compensation partial
    float* cp = (kStep && a.comp_part) ? a.comp_part + ((size_t)u * a.part_count + nc) * G * (D + 2) : nullptr;
    if (X == 0) {  // empty sequence: neutral partials
        for (int g = tid; g < G; g += kThreads) {
            pp[2 * g] = -INFINITY;
            pp[2 * g + 1] = 0.0f;
        }
        if (cp)
            for (int idx = tid; idx < G * (D + 2); idx += kThreads) cp[idx] = (idx % (D + 2) == 0) ? -INFINITY : 0.0f;
        return;
    }
    const int b = X - 1, nb = n - b * geo.B;
    const size_t blk = (size_t)u * geo.xcap + b;
    // a length beyond max_seq_len appends nothing (row n - 1 would lie past the sized range): the unit
    // is scored over max_seq_len tokens from its stored summaries, as in the separate calls
    const bool append = kStep && a.k_new && n_raw <= geo.max_seq;
    if (append) {  // the summary reads row n - 1 from k_new / v_new; the cache row is stored at the end
        if constexpr (kStep) {
            const size_t row0 = (size_t)block_row0(geo, u, b);
            const BlockSrc src{a.Kc + row0 * D, a.Vc + row0 * D, a.k_new + (size_t)u * D, a.v_new + (size_t)u * D, nb,
                               nb - 1};
            BlockRows rows;
            load_block_rows<D>(src, 0, rows);
            store_query<D, G>(qp, a.scale, geo.r, geo.layout, ts.q, ts.Qv);  // while the rows are in flight
            block_stats_from<D>(src, rows, geo.r, geo.layout, a.kmean_w + blk * D, a.dvar_w + blk * geo.r,
                                a.vmean + blk * D, ts.bs);  // (its barriers also publish ts.q / ts.Qv)
        }
    } else {
        for (int i = tid; i < D; i += kThreads) {
            ts.bs.km[i] = a.kmean[blk * D + i];
            if constexpr (kStep) ts.bs.vm[i] = a.vmean[blk * D + i];
        }
        for (int t = tid; t < geo.r; t += kThreads) ts.bs.dv[t] = a.dvar[blk * geo.r + t];
        store_query<D, G>(qp, a.scale, geo.r, geo.layout, ts.q, ts.Qv);
        __syncthreads();
    }
    for (int g = wave; g < G; g += 4) {
        float z = 0.0f, v = 0.0f;
        for (int i = lane; i < D; i += 64) z += ts.q[g][i] * ts.bs.km[i];
        for (int t = lane; t < geo.r; t += 64) v += ts.Qv[g][t] * ts.bs.dv[t];
        z = wave_sum(z);
        v = wave_sum(v);
        if (lane == 0) {
            ts.z[g] = z;
            ts.v[g] = v;
        }
    }
    __syncthreads();
    const float lnb = logf((float)nb);
    for (int g = tid; g < G; g += kThreads) {
        const float z = ts.z[g], v = ts.v[g];
        if (a.zlog) a.zlog[((size_t)u * G + g) * a.zstride + b] = z;
        pp[2 * g] = lnb + z + kind_half(a.score_kind) * v;  // the partial of one block: max a, sum exp(a - a) = 1
        pp[2 * g + 1] = 1.0f;
        if (!a.logit_terms) a.ws_w[((size_t)u * geo.xmax() + b) * G + g] = kind_term(a.score_kind, v);
    }
    if (a.logit_terms)  // the query's group sums for the selection (r = 4)
        for (int idx = tid; idx < G * 4; idx += kThreads) a.ws_qv[(size_t)u * G * 4 + idx] = ts.Qv[idx / 4][idx % 4];
    if (cp) {
        for (int idx = tid; idx < G * D; idx += kThreads) {
            const int g = idx / D, i = idx % D;
            float* p = cp + (size_t)g * (D + 2);
            if (i == 0) {
                p[0] = lnb + ts.z[g];
                p[1] = 1.0f;
            }
            p[2 + i] = ts.bs.vm[i];
        }
    }
    if (append && wave == 0) {  // the new token's cache row
        const size_t row = (size_t)block_row0(geo, u, b) + (n - 1 - b * geo.B);
        const uint4* kn = reinterpret_cast<const uint4*>(a.k_new + (size_t)u * D);
        const uint4* vn = reinterpret_cast<const uint4*>(a.v_new + (size_t)u * D);
        for (int i = lane; i < D / 8; i += 64) {
            reinterpret_cast<uint4*>(a.Kc + row * D)[i] = kn[i];
            reinterpret_cast<uint4*>(a.Vc + row * D)[i] = vn[i];
        }
    }
}

// PMAX = bpc / 32: block slots per thread (the chunk is 32 PMAX blocks). Phase-trace slots: 0 start,
// 1 role (1 chunk, 2 last block), 2 query in LDS, 3 first slot computed, 4 every slot computed,
// 6 stores begin, 15 end.
// RV: variances per lane and block that a slot may hold, 1 (up to eight variance groups), 4 (up to 32) or D / 8. With
// more than one, a slot's variances past the lane's first are requested with its mean key too, all of them at
// once. (In a loop of dependent loads after the keys, 16 units of 1024 blocks with a variance per coordinate, 17 MB,
// took 11.0 us; so 6.9.) The registers this takes stay out of the kernels of fewer groups, where they would cost
// resident workgroups: with D / 8 also for 16 and 32 groups, 64 units of 2048 blocks (G = 8, d = 128) took 67.4 us for the
// two calls at r = 16 against 63.7 so (64.8 with the loop), 64.9 against 67.6 at r = 32. (A branch around the loads past
// the last group costs 1 to 7%: they repeat the last group instead.)
template <int D, int G, bool kStep, int PMAX, int RV>
__global__ __launch_bounds__(kThreads) void score_chunks_kernel(Geom geo, ScoreArgs a) {
    constexpr int NB = chunk_slots<PMAX>();
    static_assert(NB % 64 == 0 && NB >= 32 * PMAX, "per-block rows must cover the chunk and whole waves");
    __shared__ ChunkLds<D, G, kStep, NB> lds;
    const int units = geo.units();
    COMPKV_TRACE_START();
    const int tail = a.tail_first ? (int)blockIdx.x : (int)blockIdx.x - units * a.nchunks;
    if (tail >= 0 && tail < units) {
        COMPKV_MARK_VALUE(a.trace, 1, 2);
        score_tail<D, G, kStep>(geo, a, tail, lds.t);
        COMPKV_TRACE_END(a.trace);
        return;
    }
    COMPKV_MARK_VALUE(a.trace, 1, 1);
    const int ck = a.tail_first ? (int)blockIdx.x - units : (int)blockIdx.x;
    constexpr int NF4 = D / 32;           // float4 of the mean-key row per lane
    constexpr int LPB = D / 4;            // compensation: lanes per mean-value row (one float4 each)
    constexpr int RPS = kThreads / LPB;   // mean-value rows per workgroup step
    constexpr int VROWS = kStep ? 32 * PMAX / RPS : 1;
    ChunkShared<D, G, NB>& sh = lds.c.sh;
    auto& st = lds.c.st;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    // every chunk of unit u (like its last-block workgroup) on XCD u % kXcds, the XCD whose L2 the
    // unit's selection then reads the chunks' outputs through (the chunks' linear ids start at 0 or at
    // units, a multiple of kXcds whenever the mapping applies)
    int u, chunk;
    xcd_unit_work(ck, units, a.nchunks, u, chunk);
    const int bseq = u / geo.hkv, h = u % geo.hkv;
    const int xmax = geo.xmax();
    const float s = a.scale;
    const int chunk0 = chunk * a.bpc;
    const int li = tid & 7, grp = tid >> 3;
    const int vli = tid % LPB, vslot = tid / LPB;
    const bool comp = kStep && a.comp_part != nullptr;  // fused step with Mean compensation (uniform)
    const float half = kind_half(a.score_kind);

    // The sequence length and the query pairs first, on their own: loads return in order per compute
    // unit, so requesting the mean keys only once the query is in LDS keeps the query (and the first
    // slots' keys) from queueing behind the mean keys of the other workgroups on the CU. Then per slot
    // the mean key and first variance group (the mean values follow once the keys are consumed, which
    // halves the registers held). Block ids past the allocated range load block 0 of the unit; values
    // of blocks that turn out invalid are never used (every result below is selected by validity).
    const int n_raw = a.seq_lens[bseq];
    const uint16_t* qh = a.q + ((size_t)bseq * geo.hq + (size_t)h * G) * D;
    QueryPairs<D, G> qp;
    load_query_pairs<D, G>(qh, geo.layout, qp);
    store_query<D, G>(qp, s, geo.r, geo.layout, sh.q, sh.Qv);
    const int n = clamp_len(n_raw, geo.max_seq);
    const int X = (n + geo.B - 1) / geo.B;
    const int xs = X - 1;  // blocks [0, X - 1) are scored here (all full); the last one by the extra workgroup
    const float logB = logf((float)geo.B);
    __syncthreads();
    COMPKV_MARK(a.trace, 2);  // the query in LDS
    // a chunk past the sequence's full blocks (workgroup-uniform): neutral partials, nothing read (with the
    // clamp below, ragged batches no longer read the longest sequence's blocks for every unit: 256 units of
    // 1K-8K tokens, this launch 18.6 -> 15.0 us)
    if (chunk0 >= xs) {
        float* pp = a.ws_part + ((size_t)u * (a.nchunks + 1) + chunk) * G * 2;
        for (int g = tid; g < G; g += kThreads) {
            pp[2 * g] = -INFINITY;
            pp[2 * g + 1] = 0.0f;
        }
        if (comp) {
            float* cp = a.comp_part + ((size_t)u * a.part_count + chunk) * G * (D + 2);
            for (int idx = tid; idx < G * (D + 2); idx += kThreads) cp[idx] = (idx % (D + 2) == 0) ? -INFINITY : 0.0f;
        }
        COMPKV_TRACE_END(a.trace);
        return;
    }
    // a rolling window of two slots: slot p + 2 is requested once slot p is computed
    float4 kv[2][NF4];
    float dvw[2][RV];
    auto issue = [&](int p, int w) {
        const int b = chunk0 + p * 32 + grp;
        const size_t blk = (size_t)u * geo.xcap + (b < xs ? b : chunk0);
        const float4* kp = reinterpret_cast<const float4*>(a.kmean + blk * D);
#pragma unroll
        for (int m = 0; m < NF4; ++m) kv[w][m] = kp[li + 8 * m];
#pragma unroll
        for (int j = 0; j < RV; ++j) dvw[w][j] = a.dvar[blk * geo.r + min(li + 8 * j, geo.r - 1)];
    };
    issue(0, 0);
    if (PMAX > 1) issue(1, 1);
    float4 vrow[VROWS];

    // slot by slot, in the order the slots' loads return: the projected variances (the lead lane of
    // each block keeps them in LDS), then the block-mean logits one pair of heads at a time, the pair's
    // query slice read from LDS into registers
    float qv[G];
#pragma unroll
    for (int g = 0; g < G; ++g) qv[g] = li < geo.r ? sh.Qv[g][li] : 0.0f;
    constexpr int GB = G < 2 ? G : 2;
#pragma unroll
    for (int p = 0; p < PMAX; ++p) {
        const int w = p & 1;
        const int lb = p * 32 + grp;
        const int b = chunk0 + lb;
        const bool valid = b < xs;
        const float lnb = valid ? logB : 0.0f;
        float v[G];
#pragma unroll
        for (int g = 0; g < G; ++g) {
            v[g] = qv[g] * dvw[w][0];
            // the rounded product, not fused into the sum over the lanes: the other launch shapes' bits
            __asm__("" : "+v"(v[g]));
        }
        if constexpr (RV > 1) {
#pragma unroll
            for (int j = 1; j < RV; ++j) {
                if (8 * j >= geo.r) break;  // workgroup-uniform (r is a multiple of eight here)
#pragma unroll
                for (int g = 0; g < G; ++g) v[g] = __builtin_fmaf(sh.Qv[g][li + 8 * j], dvw[w][j], v[g]);
            }
        }
#pragma unroll
        for (int g = 0; g < G; ++g) {
            v[g] = sum8_lead(v[g]);
            if (li == 0) sh.v[g][lb] = v[g];
        }
#pragma unroll 1
        for (int g0 = 0; g0 < G; g0 += GB) {
            float4 qq[GB][NF4];
#pragma unroll
            for (int gb = 0; gb < GB; ++gb)
#pragma unroll
                for (int m = 0; m < NF4; ++m) qq[gb][m] = *reinterpret_cast<const float4*>(&sh.q[g0 + gb][4 * (li + 8 * m)]);
#pragma unroll
            for (int gb = 0; gb < GB; ++gb) {
                float z = 0.0f;
#pragma unroll
                for (int m = 0; m < NF4; ++m)
                    z += qq[gb][m].x * kv[w][m].x + qq[gb][m].y * kv[w][m].y + qq[gb][m].z * kv[w][m].z +
                         qq[gb][m].w * kv[w][m].w;
                z = sum8_lead(z);
                if (li == 0) {
                    const int g = g0 + gb;
                    sh.z[g][lb] = z;
                    if constexpr (kStep) st.cw[g][lb] = valid ? lnb + z : -INFINITY;  // pseudo-logit
                }
            }
        }
        if (p + 2 < PMAX) issue(p + 2, w);
        if (p == 0) COMPKV_MARK(a.trace, 3);  // the first slot computed
    }
    COMPKV_MARK(a.trace, 4);  // every slot computed
    if (comp) {  // mean-value rows, requested once the mean keys are consumed
        const float4* vm = reinterpret_cast<const float4*>(a.vmean + (size_t)u * geo.xcap * D) + vli;
#pragma unroll
        for (int k = 0; k < VROWS; ++k) {
            const int b = chunk0 + vslot + k * RPS;
            vrow[k] = vm[(size_t)(b < xs ? b : chunk0) * (D / 4)];
        }
    }
    __syncthreads();
    // log weight a = log|b| + zbar + half * sig2 of valid block lb of the chunk
    auto logw = [&](int g, int lb) {  // (every block of a chunk is full: |b| = B)
        return logB + sh.z[g][lb] + half * sh.v[g][lb];
    };
    // the chunk's per-head max and sum of exp(a - max) (and, fused, of the pseudo-logits)
    const int nvalid = max(0, min(a.bpc, xs - chunk0));
    for (int g = wave; g < G; g += 4) {
        float av[NB / 64];
        float m = -INFINITY;
#pragma unroll
        for (int k = 0; k < NB / 64; ++k) {
            const int lb = lane + 64 * k;
            av[k] = lb < nvalid ? logw(g, lb) : -INFINITY;
            m = fmaxf(m, av[k]);
        }
        m = wave_max(m);
        float ssum = 0.0f;
        if (m != -INFINITY) {
#pragma unroll
            for (int k = 0; k < NB / 64; ++k) ssum += (av[k] == -INFINITY) ? 0.0f : expf(av[k] - m);
        }
        ssum = wave_sum(ssum);
        if (lane == 0) {
            sh.m[g] = m;
            float* pp = a.ws_part + (((size_t)u * (a.nchunks + 1) + chunk) * G + g) * 2;
            pp[0] = m;
            pp[1] = ssum;
        }
        if constexpr (kStep) if (comp) {
            float cv[NB / 64];
            float cm = -INFINITY;
#pragma unroll
            for (int k = 0; k < NB / 64; ++k) {
                const int lb = lane + 64 * k;
                cv[k] = lb < nvalid ? st.cw[g][lb] : -INFINITY;
                cm = fmaxf(cm, cv[k]);
            }
            cm = wave_max(cm);
            float csum = 0.0f;
#pragma unroll
            for (int k = 0; k < NB / 64; ++k) {
                const int lb = lane + 64 * k;
                const float wv = (cv[k] == -INFINITY) ? 0.0f : __expf(cv[k] - cm);
                st.cw[g][lb] = wv;
                csum += wv;
            }
            csum = wave_sum(csum);
            if (lane == 0) {
                st.cm[g] = cm;
                st.cl[g] = csum;
            }
        }
    }
    __syncthreads();
    COMPKV_MARK(a.trace, 6);  // the chunk's partials formed: stores
    // coalesced stores: block logits [g][b] (when requested) and score terms [b][g]
    for (int idx = tid; a.zlog && idx < G * nvalid; idx += kThreads) {
        const int g = idx / nvalid, lb = idx % nvalid;
        a.zlog[((size_t)u * G + g) * a.zstride + chunk0 + lb] = sh.z[g][lb];
    }
    for (int idx = tid; !a.logit_terms && idx < G * nvalid; idx += kThreads) {
        const int lb = idx / G, g = idx % G;
        a.ws_w[((size_t)u * xmax + chunk0 + lb) * G + g] =
            expf(logw(g, lb) - sh.m[g]) * kind_term(a.score_kind, sh.v[g][lb]);
    }
    if constexpr (kStep) if (comp) {
        // weighted mean values; lane vli of a row slot holds coordinates 4 vli .. 4 vli + 3
        float acc[G][4];
#pragma unroll
        for (int g = 0; g < G; ++g) acc[g][0] = acc[g][1] = acc[g][2] = acc[g][3] = 0.0f;
#pragma unroll
        for (int k = 0; k < VROWS; ++k) {
            const int lb = vslot + k * RPS;
            if (lb < nvalid) {
#pragma unroll
                for (int g = 0; g < G; ++g) {
                    const float wv = st.cw[g][lb];
                    acc[g][0] += wv * vrow[k].x;
                    acc[g][1] += wv * vrow[k].y;
                    acc[g][2] += wv * vrow[k].z;
                    acc[g][3] += wv * vrow[k].w;
                }
            }
        }
#pragma unroll
        for (int off = LPB; off < 64; off <<= 1)
#pragma unroll
            for (int g = 0; g < G; ++g)
#pragma unroll
                for (int e = 0; e < 4; ++e) acc[g][e] = xor_add(acc[g][e], off);
        if (lane < LPB) {
#pragma unroll
            for (int g = 0; g < G; ++g)
#pragma unroll
                for (int e = 0; e < 4; ++e) st.acc[wave][g][4 * vli + e] = acc[g][e];
        }
        __syncthreads();
        float* cp = a.comp_part + ((size_t)u * a.part_count + chunk) * G * (D + 2);
        for (int idx = tid; idx < G * D; idx += kThreads) {
            const int g = idx / D, i = idx % D;
            float* p = cp + (size_t)g * (D + 2);
            if (i == 0) {
                p[0] = st.cm[g];
                p[1] = st.cl[g];
            }
            p[2 + i] = st.acc[0][g][i] + st.acc[1][g][i] + st.acc[2][g][i] + st.acc[3][g][i];
        }
    }
    COMPKV_TRACE_END(a.trace);
}

template <int G, bool kLogits = false>
__global__ __launch_bounds__(kFinThreads) void select_finalize_kernel(Geom geo, ScoreArgs a) {
    __shared__ FinalShared sh;
    extern __shared__ float dyn[];
    const int u = blockIdx.x;
    finalize_select<G, false, kFinThreads, kLogits ? 4 : kKeysPerThread, kLogits>(
        geo, a, u, sh, dyn, a.sel + (size_t)u * a.K, a.n_sel + u, true);
}


// ---------------------------------------------------------------- one workgroup per unit
// For units with few blocks (G * xmax <= kUnitTerms) one 1024-thread workgroup per unit refreshes the
// active block (fused step), forms every block's block-mean logits, projected variances and log
// weight estimates (kept in LDS), the per-head log normalizers over every block, the scores and the
// selection: one launch, no partials. The summaries are read in batches of passes of 128 blocks (8
// lanes per block, as in the chunk kernel), each batch's loads issued before its arithmetic.
constexpr int kUnitBatch = 2;  // passes whose summaries a thread requests at once

template <int D, int G>
struct UnitShared {
    float q[G][D];
    float Qv[G][D];
    BlockStatsLds<D> bs;
    float lse[G];
};

template <int D, int G, bool kStep>
__global__ __launch_bounds__(kFinThreads) void unit_select_kernel(Geom geo, ScoreArgs a) {
    constexpr int FT = kFinThreads, KPT = kKeysPerThread, NF4 = D / 32, PB = kUnitBatch;
    constexpr int GPP = FT / 8;  // blocks per pass
    __shared__ FinalShared sh;
    __shared__ UnitShared<D, G> us;
    extern __shared__ float dyn[];  // [xmax][G] log weights (later the key bits), [xmax][G] projected variances
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int u = blockIdx.x, bseq = u / geo.hkv, h = u % geo.hkv;
    const int xmax = geo.xmax();
    const int li = tid & 7, grp = tid >> 3;
    float* A = dyn;
    float* Vp = dyn + (size_t)xmax * G;
    const float s = a.scale;

    // loads in the order of their use: query pairs, the refreshed block's rows, the first batch
    const uint16_t* qh = a.q + ((size_t)bseq * geo.hq + (size_t)h * G) * D;
    QueryPairs<D, G> qp;
    if (wave < 4) load_query_pairs<D, G>(qh, geo.layout, qp);
    __asm__ volatile("" ::: "memory");
    const int n_raw = a.seq_lens[bseq];
    const int n = clamp_len(n_raw, geo.max_seq);
    const int X = (n + geo.B - 1) / geo.B;
    const int npass = (X + GPP - 1) / GPP;
    // workgroup-uniform; a length beyond max_seq_len appends nothing (as in the chunked path)
    const bool refresh = kStep && a.k_new && X >= 1 && n_raw <= geo.max_seq;
    const int lastb = X - 1;
    const size_t blk_last = (size_t)u * geo.xcap + (lastb >= 0 ? lastb : 0);
    BlockSrc src{};
    BlockRows rows;
    if (refresh) {
        const size_t row0 = (size_t)block_row0(geo, u, lastb);
        const int nb = n - lastb * geo.B;
        src = BlockSrc{a.Kc + row0 * D, a.Vc + row0 * D, a.k_new + (size_t)u * D, a.v_new + (size_t)u * D, nb, nb - 1};
        if (wave < 4) load_block_rows<D>(src, 0, rows);
    }
    float4 kv[PB][NF4];
    float dv0[PB];
    auto issue = [&](int p0) {  // branch-free: ids past xmax load block 0, unused
#pragma unroll
        for (int p = 0; p < PB; ++p) {
            const int b = (p0 + p) * GPP + grp;
            const size_t blk = (size_t)u * geo.xcap + (b < xmax ? b : 0);
            const float4* kp = reinterpret_cast<const float4*>(a.kmean + blk * D);
#pragma unroll
            for (int m = 0; m < NF4; ++m) kv[p][m] = kp[li + 8 * m];
            dv0[p] = a.dvar[blk * geo.r + min(li, geo.r - 1)];
        }
    };
    issue(0);
    if (wave < 4) store_query<D, G>(qp, s, geo.r, geo.layout, us.q, us.Qv);
    select_init(sh);
    if (refresh)  // (its barriers also publish the query)
        block_stats_from<D>(src, rows, geo.r, geo.layout, a.kmean_w + blk_last * D, a.dvar_w + blk_last * geo.r,
                            a.vmean + blk_last * D, us.bs, wave < 4);
    else
        __syncthreads();

    // every block: zbar, sig2 and a = log|b| + zbar + sig2 / 2 per head. A block's sig2 goes to LDS
    // first; the lane that wrote it reads it back for a.
    constexpr int GB = G < 2 ? G : 2;
    float qv0[G];
#pragma unroll
    for (int g = 0; g < G; ++g) qv0[g] = li < geo.r ? us.Qv[g][li] : 0.0f;
    for (int p0 = 0; p0 < npass; p0 += PB) {  // workgroup-uniform
        if (p0 > 0) issue(p0);
        if (refresh) {
#pragma unroll
            for (int p = 0; p < PB; ++p) {
                if ((p0 + p) * GPP + grp == lastb) {  // the refreshed summary
#pragma unroll
                    for (int m = 0; m < NF4; ++m) kv[p][m] = *reinterpret_cast<const float4*>(&us.bs.km[4 * (li + 8 * m)]);
                    dv0[p] = us.bs.dv[min(li, geo.r - 1)];
                }
            }
        }
#pragma unroll
        for (int p = 0; p < PB; ++p) {
            const int b = (p0 + p) * GPP + grp;
            const bool valid = b < X;
            float v[G];
#pragma unroll
            for (int g = 0; g < G; ++g) v[g] = qv0[g] * dv0[p];
            if (geo.r > 8 && valid) {
                const size_t blk = (size_t)u * geo.xcap + b;
                for (int t = li + 8; t < geo.r; t += 8) {
                    const float dv = (refresh && b == lastb) ? us.bs.dv[t] : a.dvar[blk * geo.r + t];
#pragma unroll
                    for (int g = 0; g < G; ++g) v[g] += us.Qv[g][t] * dv;
                }
            }
#pragma unroll
            for (int g = 0; g < G; ++g) {
                v[g] = sum8_lead(v[g]);
                if (li == 0 && valid) Vp[b * G + g] = v[g];
            }
        }
#pragma unroll 1
        for (int g0 = 0; g0 < G; g0 += GB) {  // (not unrolled: one head pair's query in registers at a time)
            float4 qq[GB][NF4];
#pragma unroll
            for (int gb = 0; gb < GB; ++gb)
#pragma unroll
                for (int m = 0; m < NF4; ++m) qq[gb][m] = *reinterpret_cast<const float4*>(&us.q[g0 + gb][4 * (li + 8 * m)]);
#pragma unroll
            for (int p = 0; p < PB; ++p) {
                const int b = (p0 + p) * GPP + grp;
                const bool valid = b < X;
#pragma unroll
                for (int gb = 0; gb < GB; ++gb) {
                    float z = 0.0f;
#pragma unroll
                    for (int m = 0; m < NF4; ++m)
                        z += qq[gb][m].x * kv[p][m].x + qq[gb][m].y * kv[p][m].y + qq[gb][m].z * kv[p][m].z +
                             qq[gb][m].w * kv[p][m].w;
                    z = sum8_lead(z);
                    if (li == 0 && valid) {
                        const int g = g0 + gb;
                        const float lnb = logf((float)min(geo.B, n - b * geo.B));
                        A[b * G + g] = lnb + z + kind_half(a.score_kind) * Vp[b * G + g];
                        if (a.zlog) a.zlog[((size_t)u * G + g) * a.zstride + b] = z;
                    }
                }
            }
        }
    }
    if (refresh && wave == 4) {  // the new token's cache row (the refresh read it from k_new / v_new)
        const size_t row = (size_t)block_row0(geo, u, lastb) + (n - 1 - lastb * geo.B);
        const uint4* kn = reinterpret_cast<const uint4*>(a.k_new + (size_t)u * D);
        const uint4* vn = reinterpret_cast<const uint4*>(a.v_new + (size_t)u * D);
        for (int i = lane; i < D / 8; i += 64) {
            reinterpret_cast<uint4*>(a.Kc + row * D)[i] = kn[i];
            reinterpret_cast<uint4*>(a.Vc + row * D)[i] = vn[i];
        }
    }
    __syncthreads();
    // wave g: head g's log normalizer over every block
    if (wave < G) {
        const int g = wave;
        float m = -INFINITY;
        for (int b = lane; b < X; b += 64) m = fmaxf(m, A[b * G + g]);
        m = wave_max(m);
        float l = 0.0f;
        for (int b = lane; b < X; b += 64) l += expf(A[b * G + g] - m);
        l = wave_sum(l);
        if (lane == 0) us.lse[g] = m + logf(l);
    }
    __syncthreads();
    // scores and keys; thread t holds blocks t + 1024k
    unsigned long long ck[KPT];
    uint32_t mx = 0u;
#pragma unroll
    for (int k = 0; k < KPT; ++k) {
        const int b = tid + k * FT;
        ck[k] = 0ull;
        if (b < X) {
            float S = 0.0f;
#pragma unroll
            for (int g = 0; g < G; ++g) S += expf(A[b * G + g] - us.lse[g]) * kind_term(a.score_kind, Vp[b * G + g]);
            if (a.scores) a.scores[(size_t)u * geo.xcap + b] = S;
            if (!mandatory(b, X, a.n_sink, a.n_recent)) {
                ck[k] = ((unsigned long long)__float_as_uint(S) << 32) | (0xFFFFFFFFu - (uint32_t)b);
                mx = max(mx, __float_as_uint(S));
            }
        }
    }
    // (the key bits of the radix path overwrite the log weights, which every thread has read by then)
    const SelectCtx sc = make_select_ctx(X, a.K, a.n_sink, a.n_recent, a.sel + (size_t)u * a.K, a.n_sel + u,
                                         reinterpret_cast<uint32_t*>(A));
    if (select_fast<KPT>(sc, ck, mx, sh)) return;
    __syncthreads();
    select_radix(sc, sh);
}

template <int D, int G, bool kStep, int PMAX, int RV>
void launch_chunks_p(const Geom& g, ScoreArgs a, hipStream_t s) {
    const int grid = (a.nchunks + 1) * g.units();
    a.tail_first = grid <= resident_slots<score_chunks_kernel<D, G, kStep, PMAX, RV>>();
    score_chunks_kernel<D, G, kStep, PMAX, RV><<<dim3(grid), kThreads, 0, s>>>(g, a);
}

template <int D, int G, bool kStep, int RV>
void launch_chunks_r(const Geom& g, const ScoreArgs& a, hipStream_t s) {
    switch (a.bpc / 32) {
        case 1: launch_chunks_p<D, G, kStep, 1, RV>(g, a, s); break;
        case 2: launch_chunks_p<D, G, kStep, 2, RV>(g, a, s); break;
        default: launch_chunks_p<D, G, kStep, 4, RV>(g, a, s); break;
    }
}

template <int D, int G, bool kStep>
void launch_chunks(const Geom& g, const ScoreArgs& a, hipStream_t s) {
    if (g.r <= 8)
        launch_chunks_r<D, G, kStep, 1>(g, a, s);
    else if (g.r <= 32)
        launch_chunks_r<D, G, kStep, 4>(g, a, s);
    else
        launch_chunks_r<D, G, kStep, D / 8>(g, a, s);
}

template <int D, int G>
hipError_t launch_pair(const Geom& g, const ScoreArgs& a, hipStream_t s) {
    if (a.one_group) {
        const size_t dyn = (size_t)2 * g.xmax() * G * sizeof(float);
        if (a.k_new)
            unit_select_kernel<D, G, true><<<dim3(g.units()), kFinThreads, dyn, s>>>(g, a);
        else
            unit_select_kernel<D, G, false><<<dim3(g.units()), kFinThreads, dyn, s>>>(g, a);
        return hipGetLastError();
    }
    if (a.comp_part || a.k_new)  // fused step: the refresh and / or the compensation partials
        launch_chunks<D, G, true>(g, a, s);
    else
        launch_chunks<D, G, false>(g, a, s);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess || a.chunks_only) return e;
    if constexpr (G == 8) {
        if (a.logit_terms) {
            select_finalize_kernel<G, true><<<dim3(g.units()), kFinThreads, finalize_dyn_lds(g, a), s>>>(g, a);
            return hipGetLastError();
        }
    }
    select_finalize_kernel<G><<<dim3(g.units()), kFinThreads, finalize_dyn_lds(g, a), s>>>(g, a);
    return hipGetLastError();
}

template <int D>
hipError_t dispatch_g(const Geom& g, const ScoreArgs& a, hipStream_t s) {
    switch (g.G) {
        case 1: return launch_pair<D, 1>(g, a, s);
        case 2: return launch_pair<D, 2>(g, a, s);
        case 4: return launch_pair<D, 4>(g, a, s);
        case 8: return launch_pair<D, 8>(g, a, s);
        default: return hipErrorInvalidValue;
    }
}

}  // namespace

int select_max_bpc() { return kBpcMax; }

// the selection's logit-terms input (ScoreArgs::logit_terms) within its limits
bool logit_terms_ok(const Geom& g, const ScoreArgs& a) {
    return !a.logit_terms || (g.r == 4 && g.G == 8 && g.xmax() <= 4 * kFinThreads && a.zlog && a.ws_qv);
}

int select_one_group_terms() { return kUnitTerms; }
int select_one_group_auto_blocks() { return kUnitBatch * kFinThreads / 8; }
int select_max_chunk_heads() { return (int)(kDynBudget / (2 * sizeof(float))); }

hipError_t launch_score_select(const Geom& g, ScoreArgs a, hipStream_t s) {
    if (!logit_terms_ok(g, a) || (a.logit_terms && a.one_group)) return hipErrorInvalidValue;
    if (a.one_group) {
        if (g.G * g.xmax() > kUnitTerms) return hipErrorInvalidValue;
        return g.D == 128 ? dispatch_g<128>(g, a, s) : dispatch_g<64>(g, a, s);
    }
    if (a.bpc != 32 && a.bpc != 64 && a.bpc != 128) return hipErrorInvalidValue;
    a.keys_in_lds = 0;
    a.keys_in_lds = finalize_dyn_lds(g, a) + (size_t)g.xmax() * sizeof(float) <= kDynBudget;
    if (finalize_dyn_lds(g, a) > kDynBudget) return hipErrorInvalidValue;
    return g.D == 128 ? dispatch_g<128>(g, a, s) : dispatch_g<64>(g, a, s);
}

}  // namespace compkv
