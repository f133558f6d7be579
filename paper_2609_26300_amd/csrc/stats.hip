// stats.hip -- block summaries: prefill build and streaming append (Sections 4.1, 4.2; Appendix E.1).
//
// The prefill strides over every (unit, block): one wave per block up to 64 rows at d = 128 (from 33 rows on
// while the blocks occupy every wave of a round), else one workgroup (wg_block_stats, block_stats.h). The append
// recomputes each unit's active block with the workgroup routine after storing the new row, like the fused decode
// step. Wave and workgroup add in the same order, so an appended block's summary is bit-identical to the prefill one.
#include "block_stats.h"

namespace compkv {
namespace {

// Grid-stride over (unit, block); the workgroup summarizes one block per iteration and requests the
// next block's rows before computing the current one.
template <int D>
__global__ __launch_bounds__(kThreads) void build_stats_kernel(Geom g, StatsArgs a) {
    __shared__ BlockStatsLds<D> L;
    const int xmax = g.xmax();
    const int total = xmax * g.units();
    struct Item {
        BlockSrc src;
        size_t blk;
        bool valid;
    };
    auto item = [&](int flat) {
        Item it{};
        it.valid = false;
        if (flat >= total) return it;
        const int u = flat / xmax, b = flat % xmax;
        const int n = clamp_len(a.seq_lens[u / g.hkv], g.max_seq);
        if (b >= (n + g.B - 1) / g.B) return it;
        const size_t row0 = (size_t)block_row0(g, u, b);
        it.src = BlockSrc{a.K + row0 * D, a.V + row0 * D, nullptr, nullptr, min(g.B, n - b * g.B), -1};
        it.blk = (size_t)u * g.xcap + b;
        it.valid = true;
        return it;
    };
    int flat = blockIdx.x;
    Item cur = item(flat);
    BlockRows rc;
    if (cur.valid) load_block_rows<D>(cur.src, 0, rc);
    while (flat < total) {  // workgroup-uniform
        const int nf = flat + gridDim.x;
        const Item nxt = item(nf);
        BlockRows rn;
        if (nxt.valid) load_block_rows<D>(nxt.src, 0, rn);
        if (cur.valid)
            block_stats_from<D>(cur.src, rc, g.r, g.layout, a.kmean + cur.blk * D, a.dvar + cur.blk * g.r,
                                a.vmean + cur.blk * D, L);
        cur = nxt;
        rc = rn;
        flat = nf;
    }
}

// Blocks of at most wave_stats_max_rows<D>(NS) rows: each wave summarizes whole blocks on its own (no
// barrier, no LDS; bit-identical to the workgroup routine), consecutive waves taking consecutive blocks.
// HBM-bound, with the vector ALUs ~40% busy: the wave holds the block's keys (needed twice) and its values, VS
// steps at a time; the next block's values are requested as soon as this block's are added and its keys as
// soon as the squared deviations are, so loads stay in flight while the wave computes (the registers are loaded in
// place). With the masks as factors, one butterfly per sum and the exact reciprocal of a power-of-two count a
// block takes 890 vector instructions. One layer of 32K tokens x 8 KV heads, d = 128, blocks of 32: 39.1 -> 27.6 us
// (143 MB, 5.2 TB/s); 128K x 4: 490 -> 443 us (5.2 TB/s); 131072 blocks of 16: 469 -> 216 us, at d = 64 516 -> 157.
// The test for sums that are not finite (partly filled blocks alone) costs up to 3%; clearing each row past a block
// instead cost up to 12%. (Five workgroups per CU asked for: without it the recomputation after the loop takes the
// small form's registers past that.)
// After a wave's last block its first row is requested once more, unused, so that no branch lies around the loads; with
// the whole block requested again a build of 2048 blocks took 11.9 us against 10.4 and one of 32K from host memory 3.02 ms
// against 2.48.
template <int D, int NS, int VS>
__global__ __launch_bounds__(kThreads, NS == 1 ? 5 : 2) void build_stats_wave_kernel(Geom g, StatsArgs a) {
    constexpr int WPG = kThreads / 64, LPR = D / 8;
    constexpr int kRows = wave_stats_max_rows<D>(NS);
    static_assert(NS % VS == 0, "whole batches of values");
    const int lane = threadIdx.x & 63, ro = lane / LPR, li = lane % LPR;
    const int xmax = g.xmax();
    const int total = xmax * g.units();
    const int nwaves = gridDim.x * WPG;
    struct Item {
        size_t row0, blk;
        int nb;  // 0: no block (past the sequence, or past the last)
    };
    // (a wave's index in a scalar register: the whole item is wave-uniform)
    const int first = blockIdx.x * WPG + __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    int flat = first;
    bool redo = false;
    auto next_item = [&]() {  // the wave's next block within its sequence
        for (; flat < total; flat += nwaves) {
            const int u = flat / xmax, b = flat - u * xmax;
            const int n = clamp_len(load_uniform(a.seq_lens + u / g.hkv), g.max_seq);
            if (b * g.B < n) {
                const size_t row0 = (size_t)__builtin_amdgcn_readfirstlane(block_row0(g, u, b));
                flat += nwaves;
                return Item{row0, (size_t)u * g.xcap + b, min(g.B, n - b * g.B)};
            }
        }
        return Item{0, 0, 0};
    };
    Item cur = next_item();
    if (cur.nb == 0) return;
    WaveRows<NS> K;
    WaveRows<VS> V;
    load_wave_rows<D, VS>(a.V + cur.row0 * D, cur.nb, 0, V);
    load_wave_rows<D, NS>(a.K + cur.row0 * D, cur.nb, 0, K);
    while (true) {
        Item nxt = next_item();
        const bool more = nxt.nb != 0;
        if (!more) nxt = Item{cur.row0, cur.blk, 1};  // (its first row once more, unused)
        const int nb = cur.nb;
        float s[4][8], mk[8], t[8];
        zero_sums(s);
#pragma unroll
        for (int s0 = 0; s0 < NS; s0 += VS) {
            add_wave_rows<D, VS, false>(V, nb, s0, mk, s);
            __builtin_amdgcn_sched_barrier(0);  // (the phases in order: nothing hoisted into more registers)
            if (s0 + VS < NS)
                load_wave_rows<D, VS>(a.V + cur.row0 * D, nb, s0 + VS, V);
            else
                load_wave_rows<D, VS>(a.V + nxt.row0 * D, nxt.nb, 0, V);
        }
        total_wave_rows<D>(s, t);
        if (nb < kRows) redo |= any_not_finite(t);
        divide8(t, nb);
        if (ro == 0) {
            float4* vo = reinterpret_cast<float4*>(a.vmean + cur.blk * D + li * 8);
            vo[0] = make_float4(t[0], t[1], t[2], t[3]);
            vo[1] = make_float4(t[4], t[5], t[6], t[7]);
        }
        __builtin_amdgcn_sched_barrier(0);
        zero_sums(s);
        add_wave_rows<D, NS, false>(K, nb, 0, mk, s);
        total_wave_rows<D>(s, mk);
        divide8(mk, nb);
        if (ro == 0) {
            float4* ko = reinterpret_cast<float4*>(a.kmean + cur.blk * D + li * 8);
            ko[0] = make_float4(mk[0], mk[1], mk[2], mk[3]);
            ko[1] = make_float4(mk[4], mk[5], mk[6], mk[7]);
        }
        pin_rows(K);
        __builtin_amdgcn_sched_barrier(0);
        zero_sums(s);
        add_wave_rows<D, NS, true>(K, nb, 0, mk, s);
        __builtin_amdgcn_sched_barrier(0);
        load_wave_rows<D, NS>(a.K + nxt.row0 * D, nxt.nb, 0, K);
        total_wave_rows<D>(s, t);
        // (a mean key that is not finite leaves no squared deviation finite: this covers the keys' sums too)
        if (nb < kRows) redo |= any_not_finite(t);
        store_wave_variances<D>(t, nb, g.r, g.layout, a.dvar + cur.blk * g.r);
        if (!more) break;
        cur = nxt;
    }
    if (!redo) return;
    // some block's sums were not finite, for which a row past a block may be to blame: the wave's blocks again, from
    // their own rows alone (here, where no next block is held, so that the loop above keeps its registers)
    flat = first;
    for (cur = next_item(); cur.nb != 0; cur = next_item())
        wave_block_alone<D>(a.K + cur.row0 * D, a.V + cur.row0 * D, cur.nb, g.r, g.layout, a.kmean + cur.blk * D,
                               a.dvar + cur.blk * g.r, a.vmean + cur.blk * D);
}

// grid = (units): workgroup u recomputes block n / B with the new row n = seq_lens (before the append)
// taken from k_new / v_new, then stores that row in the cache.
template <int D>
__global__ __launch_bounds__(kThreads) void append_stats_kernel(Geom g, StatsArgs a) {
    __shared__ BlockStatsLds<D> L;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int u = blockIdx.x;
    const int n = a.seq_lens[u / g.hkv];
    if (n < 0 || n >= g.cap) return;  // workgroup-uniform
    const int blk_id = n / g.B;
    const int nb = n - blk_id * g.B + 1;
    const uint16_t* kn = a.k_new + (size_t)u * D;
    const uint16_t* vn = a.v_new + (size_t)u * D;
    const size_t row0 = (size_t)block_row0(g, u, blk_id);
    const size_t blk = (size_t)u * g.xcap + blk_id;
    wg_block_stats<D>(a.K + row0 * D, a.V + row0 * D, nb, kn, vn, nb - 1, g.r, g.layout, a.kmean + blk * D,
                      a.dvar + blk * g.r, a.vmean + blk * D, L);
    if (wave == 0) {  // the cache row (the summary above read it from k_new / v_new)
        const size_t row = row0 + (n - blk_id * g.B);
        for (int i = lane; i < D / 8; i += 64) {
            reinterpret_cast<uint4*>(a.K_out + row * D)[i] = reinterpret_cast<const uint4*>(kn)[i];
            reinterpret_cast<uint4*>(a.V_out + row * D)[i] = reinterpret_cast<const uint4*>(vn)[i];
        }
    }
}

}  // namespace

// One resident round, at most `most` workgroups per CU: the loads in flight beyond what the latency needs
// queue at the memory and slow it. Measured (MI355X, us with 1 / 2 / 3 / 4 workgroups per CU): d = 128,
// blocks of 32, 8K blocks 31.0 / 29.7 / 32.7 / 35.7, 128K blocks 432 / 448 / 463 / 467; blocks of 16, 256K
// blocks 613 / 460 / 486 / 483; d = 64, blocks of 32, 128K blocks 322 / 228 / 206 / 212; blocks of 16, 128K
// blocks 321 / 210 / 172 / 158 and 151 with 5.
template <int D, int NS, int VS>
void launch_build_wave(const Geom& g, const StatsArgs& a, int most, hipStream_t s) {
    const long long total = (long long)g.xmax() * g.units();
    const long long wgs = (total + kThreads / 64 - 1) / (kThreads / 64);
    const long long slots = resident_slots<build_stats_wave_kernel<D, NS, VS>>(kThreads, most);
    build_stats_wave_kernel<D, NS, VS><<<dim3((unsigned)(wgs < slots ? wgs : slots)), kThreads, 0, s>>>(g, a);
}

// One wave per block up to 64 rows at d = 128 (128 at d = 64), by the load steps the block needs; larger
// blocks are shared by a workgroup's four waves. So are blocks of more than 32 rows (64 at d = 64) while they are too
// few to give every wave of a round one: a wave then takes 16 rows in turn where four waves share them. Measured, us with the
// workgroup / the wave form: blocks of 64, d = 128: 64 blocks 4.9 / 8.2, 512 6.6 / 9.3, 1024 9.3 / 11.3, 2048 (a block for
// every wave) 18.4 / 16.4, 8192 58.0 / 54.1, 32768 217 / 204; blocks of 96, d = 64: 1024 8.2 / 10.7, 2048 17.2 / 16.3,
// 16384 90 / 77.
template <int D>
void launch_build_d(const Geom& g, const StatsArgs& a, hipStream_t s) {
    const int small = D == 64 ? (g.B <= 16 ? 5 : 3) : 2;
    if (g.B <= wave_stats_max_rows<D>(1)) return launch_build_wave<D, 1, 1>(g, a, small, s);
    if (g.B <= wave_stats_max_rows<D>(2)) return launch_build_wave<D, 2, 2>(g, a, 2, s);
    const long long total = (long long)g.xmax() * g.units();
    if (g.B <= wave_stats_max_rows<D>(4) &&
        total >= (long long)resident_slots<build_stats_wave_kernel<D, 4, 2>>(kThreads, 2) * (kThreads / 64))
        return launch_build_wave<D, 4, 2>(g, a, 2, s);
    const long long slots = resident_slots<build_stats_kernel<D>>();  // one resident round, grid-stride
    build_stats_kernel<D><<<dim3((unsigned)(total < slots ? total : slots)), kThreads, 0, s>>>(g, a);
}

hipError_t launch_build_stats(const Geom& g, const StatsArgs& a, hipStream_t s) {
    if (g.D == 128)
        launch_build_d<128>(g, a, s);
    else
        launch_build_d<64>(g, a, s);
    return hipGetLastError();
}

hipError_t launch_append_stats(const Geom& g, const StatsArgs& a, hipStream_t s) {
    dim3 grid(g.units());
    if (g.D == 128)
        append_stats_kernel<128><<<grid, kThreads, 0, s>>>(g, a);
    else
        append_stats_kernel<64><<<grid, kThreads, 0, s>>>(g, a);
    return hipGetLastError();
}

}  // namespace compkv
