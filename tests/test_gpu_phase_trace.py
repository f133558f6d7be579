"""The phase-trace build (libcompkv_trace.so, compkv_phase_trace_set): its fused step computes exactly what
the normal library computes, and its records are well formed (every workgroup of both launches stamped,
in order, with a known role). Its waits for selected ids can be cut short, which changes no result. The normal
library refuses both."""
import numpy as np
import pytest
import torch

import paper_2609_26300_amd as P
import paper_2609_26300_amd.binding as B
from paper_2609_26300_amd import build as lib_build
from gpu_case import TINY, Case, make_case

pytestmark = pytest.mark.gpu


def test_normal_library_refuses_the_trace():
    with pytest.raises(P.CompkvError):
        P.compkv_phase_trace_set(None, None)


@pytest.mark.parametrize("name", ["tiny_4k", "llama8b_32k", "long_16k_b8"])
def test_traced_step_matches_and_stamps_every_workgroup(name):
    c = make_case(name, "chunked_exact")
    print(f"\n[phase trace {name}]", flush=True)
    c.build_stats()
    ref = c.decode_step()
    torch.cuda.synchronize()
    rec1 = torch.zeros(1 << 18, dtype=torch.int64, device="cuda")
    rec2 = torch.zeros(1 << 18, dtype=torch.int64, device="cuda")
    saved = (B._lib, B.LIB_PATH)
    try:
        B._lib, B.LIB_PATH = None, lib_build.TRACE_LIB
        P.compkv_phase_trace_set(rec1, rec2)
        got = c.decode_step()
        torch.cuda.synchronize()
        P.compkv_phase_trace_set(None, None)
    finally:
        B._lib, B.LIB_PATH = saved
    for k in ("sel", "n_sel", "blk_logit", "out", "lse"):
        assert torch.equal(got[k], ref[k]), k
    units = c.dims.batch * c.dims.n_kv_heads
    for rec, roles in ((rec1, (1, 2)), (rec2, (1, 2))):
        r = rec.cpu().numpy().view(np.uint64).reshape(-1, 16)
        r = r[r[:, 15] != 0]
        assert len(r) >= 2 * units
        assert set(np.unique(r[:, 1]).tolist()) <= set(roles)
        assert np.all(r[:, 0] <= r[:, 15])
        for s in range(2, 14):  # every stamped phase lies between the workgroup's start and end (14 holds its placement)
            m = r[:, s] != 0
            assert np.all((r[m, s] >= r[m, 0]) & (r[m, s] <= r[m, 15])), s
    a = rec1.cpu().numpy().view(np.uint64).reshape(-1, 16)
    b = rec2.cpu().numpy().view(np.uint64).reshape(-1, 16)
    a, b = a[a[:, 15] != 0], b[b[:, 15] != 0]
    assert np.sum(a[:, 1] == 2) == units  # one last-block workgroup per unit
    assert a[:, 15].max() <= b[:, 0].min()  # the fused launch starts after the chunk launch ends


def test_normal_library_keeps_its_waits():
    with pytest.raises(P.CompkvError):
        P.compkv_select_polls_set(0)


# one-selector launches of 512 and of 1024 threads, with one and with eight heads per unit (the latter forms its score
# terms in the selection), unit counts that do not fill whole rounds of eight, empty and full sequences
@pytest.mark.parametrize("batch,heads,d,block,context,budget", [(3, (8, 2), 128, 16, 1030, 12), (1, (4, 4), 64, 1, 1024, 33),
                                                                (3, (16, 2), 64, 16, 1030, 12), (2, (8, 1), 128, 2, 2100, 600),
                                                                (1, (4, 1), 128, 4, 8200, 600), (5, (16, 2), 64, 8, 10400, 300),
                                                                (70, (8, 2), 128, 16, 1030, 12)])
@pytest.mark.parametrize("compensation", [P.COMPKV_COMP_MEAN, P.COMPKV_COMP_DROP])
def test_workers_that_stop_waiting_select_the_same(batch, heads, d, block, context, budget, compensation):
    """With no polls allowed, a worker whose ids are not posted yet (under Drop, where it has nothing to stream first,
    every one) makes the selection itself: the outputs are the same bits, and the units' words count those waits."""
    lens = ([context, 0, context - 1, 1, block] + [1 + (37 * i) % context for i in range(5, batch)])[:batch]
    c = Case(TINY.with_(batch=batch, n_q_heads=heads[0], n_kv_heads=heads[1], head_dim=d, block_size=block, context=context,
                        budget_blocks=budget, seed=62), seq_lens=lens)
    c.compensation = compensation
    c.build_stats()
    assert P.compkv_decode_step_form(c.dims, c.params())[1] >= 2  # the one-selector form
    ref = c.decode_step()
    torch.cuda.synchronize()
    units = batch * heads[1]
    waits = c.ws.view(torch.int32)[3:4 * units:4]
    saved = (B._lib, B.LIB_PATH)
    try:
        B._lib, B.LIB_PATH = None, lib_build.TRACE_LIB
        P.compkv_select_polls_set(0)
        waits.zero_()
        for _ in range(3):
            got = c.decode_step()
        torch.cuda.synchronize()
        missed = int(waits.sum())
        waits.zero_()
        P.compkv_select_polls_set(-1)
        c.decode_step()
        torch.cuda.synchronize()
        assert int(waits.sum()) == 0
    finally:
        P.compkv_select_polls_set(-1)
        B._lib, B.LIB_PATH = saved
    for k in ("sel", "n_sel", "blk_logit", "out", "lse"):
        assert torch.equal(got[k], ref[k]), k
    if compensation == P.COMPKV_COMP_DROP:
        assert missed > 0
