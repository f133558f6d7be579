// fused.hip -- the decode step's fused selection/exact launch: its two forms and their launchers. The
// scoring launch before it is in select.hip, the pieces both share in select_core.h.
#include "select_core.h"

namespace compkv {
namespace {

// ---------------------------------------------------------------- selection + exact items, fused
// Form 1 of the fused step's selection/exact launch: a one-dimensional grid of (items + n_comp) * units
// workgroups of kSxThreads threads, mapped by xcd_unit_work so that (when the units fill whole rounds
// of eight) all workgroups of unit u run on XCD u % 8. Every item workgroup of a unit repeats the unit's
// selection from the chunk partials (the same computation as select_finalize_kernel, so all of them
// hold the same ids) into LDS; item 0 also writes the selection outputs. Then the sixteen waves attend
// exactly over the item's blocks (exact.h, one 16-token tile per wave and round) and write the item's
// partial. The unit's last workgroup to arrive merges its partials (merge_unit), so the step needs no
// further launch. The launch pays off while every workgroup is resident at once (one per CU).
//
// Compensation workgroups (the fused step with Mean compensation and the chunk launch scoring only):
// the same launch also holds n_comp workgroups per unit, after the item workgroups in the grid, that
// stream the mean values of every block while the item workgroups select. Workgroup c of unit u takes
// blocks [c cb, (c + 1) cb): the pseudo-token of each (logit log|b| + zbar_b from the block logits the
// chunk launch wrote, value vmean_b), reduced to one softmax partial per head (max, sum of weights,
// weighted mean values). The exact items take their selected blocks' pseudo-tokens back out, so the
// compensation needs no selection and the mean values stream while the HBM would otherwise idle.
// threads of the fused selection/exact launch's workgroups and keys per thread
constexpr int kSxThreads = 1024;
constexpr int kSxKeys = 8192 / kSxThreads;
// mean-value rows per thread and batch of a compensation workgroup (two batches in flight: 32 KB at
// d = 128). While nearly every CU streams, that suffices for the HBM rate, and less data queued at the
// memory keeps the latency of the selections' and the exact items' loads short.
constexpr int kCompRows = 1;
// the same in the 512-thread form, where one or two workers per unit stream the mean values (64 KB in flight
// each): 256 units of up to 8K tokens, fused launch 43.1 us against 45.0 with one row
constexpr int kCompRowsSmall = 4;

// Exact attention of unit u over nblk selected blocks whose ids are in LDS (ids; -1 or an id past the
// unit's blocks contributes nothing) into decode partial `part` of the unit (device-coherent stores).
// Under Mean compensation every token's weight is p_j - p'_j (the chunk launch's block logits).
// absorb: the workgroup's compensation partial (step_compensation with kKeep) joins the stored partial.
template <int D, int G, int NW, typename Lds>
__device__ void sx_exact(const Geom& geo, const DecodeArgs& d, int u, int n, const int32_t* ids, int nblk,
                         int part, Lds& L, bool absorb = false) {
    constexpr int FT = NW * 64;
    const int tid = threadIdx.x;
    const int bseq = u / geo.hkv, h = u % geo.hkv;
    const int X = (n + geo.B - 1) / geo.B;
    TokenMap tm;
    tm.dense = false;
    tm.B = geo.B;
    tm.invB = 1.0f / (float)geo.B;
    tm.n = n;
    tm.X = X;
    tm.nblk = nblk;
    tm.sel = ids;
    tm.t0 = tm.t1 = 0;
    tm.page = tm.pg0 = 0;
    tm.invP = 0.0f;
    tm.rowbase = L.rowbase;
    for (int k = tid; k < nblk; k += FT) {
        const int b = ids[k];
        L.rowbase[k] = block_row0(geo, u, b >= 0 && b < X ? b : 0);
    }
    __syncthreads();
    float m, l;
    v4f32 acc[D / 16];
    const uint16_t* qh = d.q + ((size_t)bseq * geo.hq + (size_t)h * G) * D;
    const bool pseudo = d.neg_pseudo != 0;  // Mean: the compensation added every block's pseudo-token
    exact_tokens<D, G, NW>(tm, d.K, d.V, qh, pseudo ? d.blk_logit + (size_t)u * G * geo.xcap : nullptr, geo.xcap,
                           L.u.ex.zb, d.scale, m, l, acc);
    COMPKV_MARK(d.trace, 8);  // this wave 0's tiles attended
    constexpr int kCwStride = (int)(sizeof(L.cw[0]) / sizeof(float));
    finish_exact<D, G, NW, true>(m, l, acc, L.u.ex, d.ws_part + ((size_t)u * d.part_count + part) * G * (D + 2),
                                 absorb ? L.cm : nullptr, L.cl, &L.cw[0][0], kCwStride);
    COMPKV_MARK(d.trace, 9);  // partial stored
}

template <int D, int G, int FT, int KPT, bool kLogits = false>
__global__ __launch_bounds__(FT) void select_exact_kernel(Geom geo, ScoreArgs a, DecodeArgs d, int items) {
    constexpr int NW = FT / 64;
    using Lds = SelExactLdsT<D, G, kStepCbMax, NW>;
    __shared__ Lds L;
    extern __shared__ float dyn[];
    const int tid = threadIdx.x;
    const int units = geo.units();
    COMPKV_TRACE_START();
    int u, item;
    if ((int)blockIdx.x >= items * units) {  // a compensation workgroup (workgroup-uniform)
        COMPKV_MARK_VALUE(d.trace, 1, 2);
        int c;
        xcd_unit_work((int)blockIdx.x - items * units, units, d.n_comp, u, c);
        const int xmax = geo.xmax();
        const int c0 = min(c * d.cb, xmax), c1 = min(c0 + d.cb, xmax);
        step_compensation<D, G, kCompRows, Lds, FT>(geo, d, u, d.seq_lens[u / geo.hkv], c0, c1, L,
                                                          d.ws_part + ((size_t)u * d.part_count + c) * G * (D + 2),
                                                          [] {});
        COMPKV_MARK(d.trace, 9);
        if (d.arrive) arrive_and_merge<D, G, Lds, FT>(geo, d, u, L);
        COMPKV_TRACE_END(d.trace);
        return;
    }
    COMPKV_MARK_VALUE(d.trace, 1, 1);
    // the items of unit u all on XCD u % kXcds: the unit's selection inputs are fetched once into
    // that XCD's L2
    xcd_unit_work(blockIdx.x, units, items, u, item);
    finalize_select<G, false, FT, KPT, kLogits>(geo, a, u, L.u.fin, dyn, L.sel, &L.nsel, item == 0);
    __syncthreads();
    COMPKV_MARK(d.trace, 4);  // selected
    const int n = clamp_len(d.seq_lens[u / geo.hkv], geo.max_seq);
    const int nsel = L.nsel;
    if (item == 0) {  // the selection outputs (the ids past n_sel hold -1)
        for (int k = tid; k < a.K; k += FT) a.sel[(size_t)u * a.K + k] = L.sel[k];
        if (tid == 0) a.n_sel[u] = nsel;
    }
    const int e0 = item * d.eb;
    sx_exact<D, G, NW>(geo, d, u, n, L.sel + e0, max(0, min(d.eb, nsel - e0)), d.part_base + item, L);
    if (d.arrive) arrive_and_merge<D, G, Lds, FT>(geo, d, u, L);
    COMPKV_TRACE_END(d.trace);
}

// ---------------------------------------------------------------- selection + exact, one selector
// The same step when every workgroup of the launch is resident at once: per unit one selector and
// P - 1 workers (grid units * P, the selectors first; xcd_unit_work keeps a unit's workgroups on one
// XCD). The selector ranks the unit's blocks and posts every id slot k < K to the unit's mailbox
// (id ^ kPosted, device-coherent; the chunk launch zeroed the mailbox, and no posted value is zero),
// then attends exactly over the first eb ids. Worker w (1 .. P - 1) first streams its share of the
// mean values (compensation blocks [(w - 1) cb, w cb)), requesting its slots [w eb, (w + 1) eb) of the
// mailbox once the last mean values are in; a slot still zero is polled until posted. Then it attends exactly over
// those ids, and its compensation partial (kept in LDS) joins its exact partial: workgroup w stores partial w,
// and the unit's last workgroup of P merges the P partials. The HBM streams from the start on every CU but the
// selectors', and the selection runs once per unit.
//
// The wait depends on the selector having started, and nothing guarantees that it has: selectors come first in the
// grid, and where the units fill whole rounds of eight a unit's workgroups queue on one XCD, its selector ahead; but
// otherwise a worker may run on one XCD while its selector still queues on another, behind workgroups of another
// stream that may themselves be waiting. So the wait is bounded (d.polls), and a worker that ends it without its ids
// makes the selection itself (the same computation: the same ids): whatever else runs on the GPU and in whatever
// order workgroups start, every workgroup ends and the results are the same. The unit's timeout word counts such waits.
// Phase-trace slots (both forms of the fused launch): 0 start, 1 role (1 selects, 2 streams mean values
// first), 2 the selection's loads in, 3 keys formed, 4 selected, 5 compensation weights formed, 6 mean
// values weighed, 7 ids in hand (worker), 8 wave 0's tiles attended, 9 partial stored, 10 merges, 15 end.
constexpr uint32_t kPosted = 0x80000000u;  // mailbox value of id b: b ^ kPosted (-1 gives 0x7FFFFFFF)
constexpr int kSelPollLimit = 1 << 14;     // polls of a wait (each a memory round trip): about 10 ms

// FT: threads, 1024 (one workgroup per CU) or 512 (two per CU: short units or many of them, chosen by the host, at
// most 2048 blocks); KPT: keys per thread of the selection (xmax <= KPT FT); kLogits: a.logit_terms
template <int D, int G, int FT, int KPT, bool kLogits = false>
__global__ __launch_bounds__(FT) void select_work_kernel(Geom geo, ScoreArgs a, DecodeArgs d, int P) {
    constexpr int NW = FT / 64;
    using Lds = SelExactLdsT<D, G, kStepCbMax, NW>;
    __shared__ Lds L;
    extern __shared__ float dyn[];
    const int tid = threadIdx.x;
    const int units = geo.units();
    COMPKV_TRACE_START();
    int u, w;
    if ((int)blockIdx.x < units) {
        u = blockIdx.x;  // (XCD blockIdx % 8 = u % 8)
        w = 0;
    } else {
        xcd_unit_work((int)blockIdx.x - units, units, P - 1, u, w);
        ++w;
    }
    uint32_t* mbox = d.mailbox + (size_t)u * a.K;
    COMPKV_MARK_VALUE(d.trace, 1, w == 0 ? 1 : 2);
    // Both roles share one copy of the selection and of the exact share below (with a copy each the code was twice as long:
    // us a step, 8 units of 32K tokens 21.4 -> 20.9, 2 units of 4K 17.9 -> 17.5, 64 units of 64K (G = 8) 43.0 -> 41.9).
    bool selects = w == 0;  // (workgroup-uniform)
    bool comp = false;      // a compensation partial waits in LDS
    int n_raw = 0, nblk = 0;
    const int e0 = w * d.eb;
    if (w != 0) {
        n_raw = d.seq_lens[u / geo.hkv];
        nblk = max(0, min(d.eb, a.K - e0));  // (the ids past n_sel are -1)
        uint32_t mv = 0u;
        auto request = [&] { mv = ld_agent_u32(mbox + (tid < nblk ? e0 + tid : 0)); };
        comp = d.n_comp > 0;
        if (comp) {  // its compensation partial stays in LDS for the exact partial to absorb
            // the 512-thread form is bound by the bytes of many short sequences: equal shares of the
            // sequence's own blocks (ragged lengths: 74 -> 60 us a step at 256 units of 1K-8K tokens).
            // The 1024-thread form is bound by latency: shares of the longest sequence, whose rows are
            // requested without waiting for the length
            const int X = FT < 1024 ? (clamp_len(n_raw, geo.max_seq) + geo.B - 1) / geo.B : geo.xmax();
            const int cb = FT < 1024 ? (X + d.n_comp - 1) / d.n_comp : d.cb;
            const int c0 = min((w - 1) * cb, X), c1 = min(c0 + cb, X);
            // the slots are polled once the last mean values are requested: if the selector has posted
            // them by then, they return with those values; else they are requested once more after them
            step_compensation<D, G, (FT < 1024 ? kCompRowsSmall : kCompRows), Lds, FT, true>(
                geo, d, u, n_raw, c0, c1, L, nullptr, [&] { if (__any(mv == 0u)) request(); }, request);
        } else {
            request();
        }
        static_assert(kMaxEb <= 128, "waves 0 and 1 hold the ids");
        if (tid < 128) {
            bool missed = false;
            if (tid < nblk) {
                for (int polls = 0; mv == 0u && polls < d.polls; ++polls) {
                    __builtin_amdgcn_s_sleep(2);
                    mv = ld_agent_u32(mbox + e0 + tid);
                }
                missed = mv == 0u;
                L.sel[tid] = (int32_t)(mv ^ kPosted);
            }
            missed = __any(missed);
            if ((tid & 63) == 0) {
                L.missed[tid >> 6] = missed;
                if (missed && d.timeouts)
                    __hip_atomic_fetch_add(d.timeouts + 4 * u + 3, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            }
        }
        __syncthreads();
        selects = (L.missed[0] | L.missed[1]) != 0;
    }
    if (selects) {
        finalize_select<G, false, FT, KPT, kLogits>(geo, a, u, L.u.fin, dyn, L.sel, &L.nsel, w == 0);
        __syncthreads();
    }
    if (w == 0) {
        COMPKV_MARK(d.trace, 4);  // selected
        for (int k = tid; k < a.K; k += FT) {
            const int32_t b = L.sel[k];
            st_agent_u32(mbox + k, (uint32_t)b ^ kPosted);
            a.sel[(size_t)u * a.K + k] = b;
        }
        if (tid == 0) a.n_sel[u] = L.nsel;
        n_raw = d.seq_lens[u / geo.hkv];
        nblk = max(0, min(d.eb, L.nsel));
    } else {
        COMPKV_MARK(d.trace, 7);  // the ids in hand
    }
    sx_exact<D, G, NW>(geo, d, u, clamp_len(n_raw, geo.max_seq), selects ? L.sel + e0 : L.sel, nblk, w, L, comp);
    if (arrive_last(d.arrive + u, P, L.last)) {
        COMPKV_MARK(d.trace, 10);  // this workgroup merges
        merge_unit<D, G, Lds, FT>(geo, d, u, L);
    }
    COMPKV_TRACE_END(d.trace);
}

template <int D, int G>
hipError_t launch_sx(const Geom& g, const ScoreArgs& a, const DecodeArgs& d, int items, hipStream_t s) {
    const dim3 grid((items + d.n_comp) * g.units());
    const size_t dyn = finalize_dyn_lds(g, a);
    if constexpr (G == 8) {
        if (a.logit_terms) {  // (at most 4096 blocks: checked by the launcher)
            if (g.xmax() <= kSxThreads)
                select_exact_kernel<D, G, kSxThreads, 1, true><<<grid, kSxThreads, dyn, s>>>(g, a, d, items);
            else
                select_exact_kernel<D, G, kSxThreads, 4, true><<<grid, kSxThreads, dyn, s>>>(g, a, d, items);
            return hipGetLastError();
        }
    }
    // keys per thread for the unit's blocks (as in launch_work)
    if (g.xmax() <= kSxThreads)
        select_exact_kernel<D, G, kSxThreads, 1><<<grid, kSxThreads, dyn, s>>>(g, a, d, items);
    else if (g.xmax() <= 4 * kSxThreads)
        select_exact_kernel<D, G, kSxThreads, 4><<<grid, kSxThreads, dyn, s>>>(g, a, d, items);
    else
        select_exact_kernel<D, G, kSxThreads, kSxKeys><<<grid, kSxThreads, dyn, s>>>(g, a, d, items);
    return hipGetLastError();
}

template <int D, int G, int FT>
hipError_t launch_work(const Geom& g, const ScoreArgs& a, const DecodeArgs& d, int P, hipStream_t s) {
    const dim3 grid(P * g.units());
    const size_t dyn = finalize_dyn_lds(g, a);
    const int xmax = g.xmax();  // (FT = 512: at most 4 FT blocks, checked by the launcher)
    constexpr int K2 = FT < 1024 ? 2 : 4;
    if constexpr (G == 8) {
        if (a.logit_terms) {  // (at most 4 FT blocks: checked by the launcher)
            if (xmax <= FT)
                select_work_kernel<D, G, FT, 1, true><<<grid, FT, dyn, s>>>(g, a, d, P);
            else if (xmax <= K2 * FT)
                select_work_kernel<D, G, FT, K2, true><<<grid, FT, dyn, s>>>(g, a, d, P);
            else
                select_work_kernel<D, G, FT, 4, true><<<grid, FT, dyn, s>>>(g, a, d, P);
            return hipGetLastError();
        }
    }
    // keys per thread for the unit's blocks: fewer loads and keys where the blocks are few
    if (xmax <= FT)
        select_work_kernel<D, G, FT, 1><<<grid, FT, dyn, s>>>(g, a, d, P);
    else if (xmax <= K2 * FT)
        select_work_kernel<D, G, FT, K2><<<grid, FT, dyn, s>>>(g, a, d, P);
    else if (FT < 1024 || xmax <= 4 * FT)
        select_work_kernel<D, G, FT, 4><<<grid, FT, dyn, s>>>(g, a, d, P);
    else if constexpr (FT == 1024)
        select_work_kernel<D, G, FT, 8><<<grid, FT, dyn, s>>>(g, a, d, P);
    return hipGetLastError();
}

template <int D, int FT>
hipError_t work_g(const Geom& g, const ScoreArgs& a, const DecodeArgs& d, int P, hipStream_t s) {
    switch (g.G) {
        case 1: return launch_work<D, 1, FT>(g, a, d, P, s);
        case 2: return launch_work<D, 2, FT>(g, a, d, P, s);
        case 4: return launch_work<D, 4, FT>(g, a, d, P, s);
        case 8: return launch_work<D, 8, FT>(g, a, d, P, s);
        default: return hipErrorInvalidValue;
    }
}

template <int D>
hipError_t sx_g(const Geom& g, const ScoreArgs& a, const DecodeArgs& d, int items, hipStream_t s) {
    switch (g.G) {
        case 1: return launch_sx<D, 1>(g, a, d, items, s);
        case 2: return launch_sx<D, 2>(g, a, d, items, s);
        case 4: return launch_sx<D, 4>(g, a, d, items, s);
        case 8: return launch_sx<D, 8>(g, a, d, items, s);
        default: return hipErrorInvalidValue;
    }
}

}  // namespace

int select_poll_limit() { return kSelPollLimit; }
int select_exact_max_budget() { return kSelLdsMax; }
int select_exact_waves() { return kSxThreads / 64; }
int select_exact_max_cb() { return kStepCbMax; }
int select_exact_merge_terms() { return kMergeMaxTerms; }

// Resident workgroups of the one-selector fused launch on the current device with `dyn` bytes of
// dynamic LDS each. The answer depends on nothing else, and every step asks it several times: each thread keeps
// the last few (a query takes about a microsecond).
template <int D, int G>
int sx_slots(size_t dyn, int threads) {
    struct Known {
        int dev, threads, slots;
        size_t dyn;
    };
    constexpr int kKnown = 8;
    static thread_local Known known[kKnown];
    static thread_local int count = 0;
    int per_cu = 0, cus = 0, dev = 0;
    if (hipGetDevice(&dev) != hipSuccess) return 0;
    for (int i = 0; i < (count < kKnown ? count : kKnown); ++i)
        if (known[i].dev == dev && known[i].threads == threads && known[i].dyn == dyn) return known[i].slots;
    if ((threads == kSxThreads
             ? hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, select_work_kernel<D, G, 1024, 8>, 1024, dyn)
             : hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, select_work_kernel<D, G, 512, 4>, 512, dyn)) !=
            hipSuccess ||
        hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess)
        return 0;
    known[count % kKnown] = {dev, threads, per_cu * cus, dyn};
    count = count + 1 < (1 << 30) ? count + 1 : kKnown;
    return per_cu * cus;
}
template <int D>
int sx_slots_d(const Geom& g, size_t dyn, int threads) {
    switch (g.G) {
        case 1: return sx_slots<D, 1>(dyn, threads);
        case 2: return sx_slots<D, 2>(dyn, threads);
        case 4: return sx_slots<D, 4>(dyn, threads);
        default: return sx_slots<D, 8>(dyn, threads);
    }
}
int select_exact_slots(const Geom& g, size_t dyn, int threads) {
    return g.D == 128 ? sx_slots_d<128>(g, dyn, threads) : sx_slots_d<64>(g, dyn, threads);
}

hipError_t launch_select_exact(const Geom& g, ScoreArgs a, const DecodeArgs& d, int items, hipStream_t s) {
    // the keys of the fast path's tie fallback stay in LDS: no workgroup writes global scratch
    a.keys_in_lds = 1;
    if (!logit_terms_ok(g, a)) return hipErrorInvalidValue;
    if (a.bpc < 1 || (a.bpc & (a.bpc - 1)) != 0 || g.xmax() > kFinThreads * kKeysPerThread || a.K > kSelLdsMax ||
        d.eb > kMaxEb ||
        finalize_dyn_lds(g, a) > kDynBudget || (d.n_comp > 0 && (d.cb < 1 || d.cb > kStepCbMax)) ||
        (long long)d.n_comp * d.cb < (d.n_comp > 0 ? g.xmax() : 0) || d.part_base + items > d.part_count ||
        (d.arrive && (d.part_count != d.n_comp + items || d.part_count * g.G > kMergeMaxTerms)))
        return hipErrorInvalidValue;
    return g.D == 128 ? sx_g<128>(g, a, d, items, s) : sx_g<64>(g, a, d, items, s);
}
hipError_t launch_select_work(const Geom& g, ScoreArgs a, const DecodeArgs& d, int P, int threads, hipStream_t s) {
    a.keys_in_lds = 1;
    if (!logit_terms_ok(g, a)) return hipErrorInvalidValue;
    const int keff = std::max(1, std::min(a.K, g.xmax()));
    if (P < 2 || a.bpc < 1 || (a.bpc & (a.bpc - 1)) != 0 || g.xmax() > kFinThreads * kKeysPerThread || a.K > kSelLdsMax ||
        d.eb < 1 || d.eb > kMaxEb || (long long)P * d.eb < keff || finalize_dyn_lds(g, a) > kDynBudget || !d.arrive ||
        !d.mailbox ||
        (d.n_comp != 0 && (d.n_comp != P - 1 || d.cb < 1 || d.cb > kStepCbMax || (long long)d.n_comp * d.cb < g.xmax())) ||
        d.part_base != 0 || d.part_count != P || d.part_count * g.G > kMergeMaxTerms)
        return hipErrorInvalidValue;
    if (threads == 512) {
        if (g.xmax() > 4 * threads) return hipErrorInvalidValue;
        return g.D == 128 ? work_g<128, 512>(g, a, d, P, s) : work_g<64, 512>(g, a, d, P, s);
    }
    if (threads != kSxThreads) return hipErrorInvalidValue;
    return g.D == 128 ? work_g<128, 1024>(g, a, d, P, s) : work_g<64, 1024>(g, a, d, P, s);
}
}  // namespace compkv
