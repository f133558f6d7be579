"""The native call path of the binding: what it passes on, what it leaves to the checks in Python."""
import ctypes

import pytest
import torch

import paper_2609_26300_amd as P
from paper_2609_26300_amd import binding as B

EINVAL = -1


def _host():
    P.library()
    if B._host_call is None:
        B._load_host()
    return B._host_call


def test_native_call_passes_words_and_status():
    """Null pointers reach the library (COMPKV_EINVAL); a count that is not the function's is refused."""
    d = P.make_dims(1, 8, 2, 128, 16, 4, 4096)
    entry = ctypes.cast(P.library().compkv_dense_decode, ctypes.c_void_p).value
    args = (ctypes.addressof(d), 0.5, 0, 0, 0, 0, 0, 0, 0, 0, 0)
    assert _host()(B._DENSE, entry, args, (None,) * 11) == EINVAL
    with pytest.raises(TypeError):
        _host()(B._DENSE, entry, args[:-1], (None,) * 10)
    with pytest.raises(TypeError):
        _host()(99, entry, args, (None,) * 11)
    with pytest.raises(TypeError):
        _host()(B._DENSE, entry, args, (None,) * 10)


@pytest.mark.parametrize("arg,spec", [
    (torch.zeros(2, 3), (torch.float32, (2, 3), False)),  # not a CUDA tensor
    (None, (torch.float32, (2, 3), False)),  # required
    ("x", (torch.float32, (2, 3), True)),
    (torch.zeros(2), True),
    ("x", None),
])
def test_native_call_leaves_the_rest_to_python(arg, spec):
    entry = ctypes.cast(P.library().compkv_dense_decode, ctypes.c_void_p).value
    assert _host()(B._DENSE, entry, (arg,), (spec,)) is None


def test_specs_follow_the_values_of_dims():
    """What a call checks depends on the dims' values, not on the object: a changed dims is another check."""
    d = P.make_dims(1, 8, 2, 128, 16, 4, 4096)
    a = B._call_spec(B._STEP, d, 16)
    d.capacity_tokens = d.max_seq_len = 8192
    b = B._call_spec(B._STEP, d, 16)
    assert a[3][1] == (1, 2, 4096, 128) and b[3][1] == (1, 2, 8192, 128)
    assert bytes(d) != bytes(P.make_dims(1, 8, 2, 128, 16, 4, 4096))


_SP = P.CompkvSelectParams(4, 1, 2, 0.1)


@pytest.mark.parametrize("call,n", [(P.compkv_build_stats, 6), (P.compkv_append_stats, 8), (P.compkv_score_select, 9),
                                    (P.compkv_sparse_decode, 10), (P.compkv_dense_decode, 7), (P.compkv_decode_step, 15),
                                    (P.compkv_decode_step_noalloc, 15)])
@pytest.mark.parametrize("dims", ["good", "no_kv_heads", "no_blocks", None])
@pytest.mark.parametrize("head", [_SP, None, 0.5, "x"])
def test_wrong_calls_fail_as_without_the_native_path(monkeypatch, call, n, dims, head):
    """Dims that form no shapes, dims and parameters that are none, tensors on the CPU: the same error, type and
    words, as from the checks in Python alone."""
    if isinstance(dims, str):
        d = P.make_dims(1, 8, 2, 128, 16, 4, 4096)
        if dims == "no_kv_heads":
            d.n_kv_heads = 0
        if dims == "no_blocks":
            d.block_size = 0
    else:
        d = dims
    takes_head = call not in (P.compkv_build_stats, P.compkv_append_stats)
    for x in (torch.zeros(1, 2, 4), None):
        args = (d, head, *[x] * n) if takes_head else (d, *[x] * n)
        got = []
        for native in (True, False):
            with monkeypatch.context() as m:
                if not native:
                    m.setattr(B, "_call", lambda *a: None)
                with pytest.raises(Exception) as e:
                    call(*args)
                got.append((e.type, str(e.value)))
        assert got[0] == got[1]


def test_only_an_integer_is_a_stream():
    """A stream that is no handle is left to the checks in Python, which refuse it."""
    assert B._raw_stream(7) == 7
    assert B._raw_stream(0.0) is None and B._raw_stream("0") is None


@pytest.mark.gpu
def test_wrong_tensors_are_named():
    """Each wrong argument of a step is refused with the binding's own message, and nothing is launched."""
    d = P.make_dims(1, 8, 2, 128, 16, 4, 256)
    z = lambda *s, dt=torch.float32: torch.zeros(*s, dtype=dt, device="cuda")
    bf, i32 = torch.bfloat16, torch.int32
    args = dict(q=z(1, 8, 128, dt=bf), k_cache=z(1, 2, 256, 128, dt=bf), v_cache=z(1, 2, 256, 128, dt=bf), k_new=None, v_new=None,
                seq_lens=torch.tensor([200], dtype=i32, device="cuda"), kmean=z(1, 2, 16, 128), dvar=z(1, 2, 16, 4),
                vmean=z(1, 2, 16, 128), sel=z(1, 2, 5, dt=i32), n_sel=z(1, 2, dt=i32), blk_logit=z(1, 2, 4, 16), scores=None,
                out=z(1, 8, 128), lse=z(1, 8), workspace=P.alloc_workspace(d, 5))
    prm = P.CompkvSelectParams(5, 1, 2, 0.1)
    P.compkv_decode_step(d, prm, **args)
    bad = dict(q=(args["q"].float(), "q must be"), k_cache=(args["k_cache"].transpose(1, 2), "k_cache must be contiguous"),
               kmean=(z(1, 2, 17, 128), "kmean must have shape"), out=(None, "out is required"),
               lse=(torch.zeros(1, 8), "lse must be a CUDA"), workspace=(None, "workspace must be"),
               k_new=(z(1, 2, 128, dt=bf), "given together"))
    for name, (value, message) in bad.items():
        with pytest.raises(P.CompkvError, match=message):
            P.compkv_decode_step(d, prm, **{**args, name: value})
    with pytest.raises(ctypes.ArgumentError):
        P.compkv_decode_step(d, prm, **args, stream=0.0)
    torch.cuda.synchronize()


def test_either_library_comes_with_the_call_path(monkeypatch, tmp_path):
    """Both builds make _host.so: the binding enters the trace library through it too."""
    from paper_2609_26300_amd import build as lib_build

    for name in ("BUILD", "LIB", "TRACE_LIB", "HOST_LIB"):
        monkeypatch.setattr(lib_build, name, str(tmp_path / name))
    for trace in (False, True):
        made = []
        monkeypatch.setattr(lib_build, "_run", lambda cmd, verbose: (made.append(cmd), open(cmd[cmd.index("-o") + 1], "w").close()))
        lib_build.build(trace=trace)
        assert any(c[0] == "g++" and any(a.endswith("host.cpp") for a in c) for c in made), trace
