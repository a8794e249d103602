"""The native marshalling accepts exactly the plain calls: what it does not accept goes to the Python binding,
whose errors are unchanged, and what it accepts gives the binding's results on the binding's stream."""
import ctypes
import types

import pytest
import torch

import paper_2608_08097_amd as P
from paper_2608_08097_amd import _lib as L

R, H, G, T, NB, B, K = 2, 2, 4, 3, 40, 16, 8


def _tensors(device):
    bf, i32 = torch.bfloat16, torch.int32
    g = torch.Generator().manual_seed(3)

    def rand(*s):
        return torch.randn(s, generator=g).to(bf).to(device)

    a, b = rand(R, H, NB, 128), rand(R, H, NB, 128)
    pages = 64
    return dict(d=P.dims(R, H * G, H, 128, B, NB), q=rand(R, T, H * G, 128), kmax=torch.maximum(a, b),
                kmin=torch.minimum(a, b), ctx=torch.tensor([NB * B, 300], dtype=i32, device=device),
                scores=torch.zeros(R, H, NB, device=device), sel=torch.zeros(R, H, K, dtype=i32, device=device),
                cnt=torch.zeros(R, H, dtype=i32, device=device),
                table=torch.arange(R * NB, dtype=i32, device=device).remainder(pages).view(R, NB).contiguous(),
                host_k=rand(pages, H, B, 128), host_v=rand(pages, H, B, 128),
                smap=torch.full((R, H, K), -1, dtype=i32, device=device),
                stamp=torch.zeros(R, H, K, dtype=i32, device=device), pool_k=torch.zeros(R, K + 1, H, B, 128, dtype=bf, device=device),
                pool_v=torch.zeros(R, K + 1, H, 128, B, dtype=bf, device=device),
                moved=torch.zeros(R, H, dtype=i32, device=device), out=torch.zeros(R, T, H * G, 128, dtype=bf, device=device),
                lse=torch.zeros(R, T, H * G, device=device),
                ws=torch.zeros(1 << 20, dtype=torch.uint8, device=device))


def _step(t, stream=None):
    d = t["d"]
    P.oasis_score_blocks(d, t["q"], T, 1, T - 1, t["kmax"], t["kmin"], t["ctx"], t["scores"], stream)
    P.oasis_select_topk(d, t["scores"], t["ctx"], K, t["sel"], t["cnt"], stream)
    P.oasis_stage_blocks(d, t["host_k"], t["host_v"], t["table"], t["ctx"], t["sel"], t["cnt"], t["scores"], K,
                         t["smap"], t["stamp"], 1, K, True, t["pool_k"], t["pool_v"], t["moved"], stream)
    P.oasis_sparse_decode_attn(d, t["q"], T, t["pool_k"], t["pool_v"], t["smap"], K, t["ctx"], None, t["out"],
                               t["lse"], t["ws"], stream)
    P.oasis_score_select(d, t["q"], T, 1, T - 1, t["kmax"], t["kmin"], t["ctx"], K, t["scores"], t["sel"], t["cnt"],
                         stream)


class _Sub(torch.Tensor):
    pass


def _args(t):
    return [ctypes.addressof(t["d"]), t["scores"], t["ctx"], K, t["sel"], t["cnt"], None]


def test_unusual_forms_are_not_accepted():
    """On the CPU: no form below may reach the library (a host tensor, other types and counts, a subclass)."""
    L.lib()
    t = _tensors("cpu")
    call = L._fast.select_topk
    assert call(*_args(t)) is None  # host tensors
    for i, x in ((1, None), (1, 5), (3, 8.0), (3, True), (3, 1 << 40), (4, t["sel"].as_subclass(_Sub)), (6, "0")):
        a = _args(t)
        a[i] = x
        assert call(*a) is None, (i, x)
    assert call(*_args(t)[:-1]) is None
    with pytest.raises(ValueError, match="scores must be a device tensor"):
        P.oasis_select_topk(t["d"], t["scores"], t["ctx"], K, t["sel"], t["cnt"], 0)


@pytest.mark.gpu
def test_checks_and_results_match_the_python_binding():
    L.lib()
    t = _tensors("cuda")
    torch.cuda.synchronize()
    for i, x in ((1, t["scores"].double()), (1, t["scores"].transpose(0, 1)), (2, t["ctx"][:1]), (4, t["sel"].long()),
                 (5, t["cnt"].cpu()), (4, t["sel"].as_subclass(_Sub))):
        a = _args(t)
        a[i] = x
        assert L._fast.select_topk(*a) is None, i
    with pytest.raises(TypeError, match="scores: dtype"):
        P.oasis_select_topk(t["d"], t["scores"].double(), t["ctx"], K, t["sel"], t["cnt"])
    with pytest.raises(ValueError, match="sel: 7 elements"):
        P.oasis_select_topk(t["d"], t["scores"], t["ctx"], K, t["sel"].view(-1)[:7], t["cnt"])
    with pytest.raises(P.OasisError, match="k = 0"):  # accepted and refused by the library
        P.oasis_select_topk(t["d"], t["scores"], t["ctx"], 0, t["sel"][:0], t["cnt"])
    outs = []
    side = torch.cuda.Stream()
    for fast, stream in ((True, None), (False, None), (True, side), (True, "current")):
        t = _tensors("cuda")
        torch.cuda.synchronize()
        keep = L._fast
        L._fast = keep if fast else None
        try:
            if stream == "current":
                with torch.cuda.stream(side):
                    _step(t)
            else:
                _step(t, stream)
        finally:
            L._fast = keep
        torch.cuda.synchronize()
        outs.append([t[n].clone() for n in ("scores", "sel", "cnt", "smap", "stamp", "pool_k", "pool_v", "moved",
                                            "out", "lse")])
    for other in outs[1:]:
        assert all(torch.equal(x, y) for x, y in zip(outs[0], other))


def _calls(t, host_k, host_v):
    """The five native functions with plain arguments, without the stream."""
    d = ctypes.addressof(t["d"])
    return {
        "score_blocks": [d, t["q"], T, 1, T - 1, t["kmax"], t["kmin"], t["ctx"], t["scores"]],
        "select_topk": [d, t["scores"], t["ctx"], K, t["sel"], t["cnt"]],
        "score_select": [d, t["q"], T, 1, T - 1, t["kmax"], t["kmin"], t["ctx"], K, t["scores"], t["sel"], t["cnt"]],
        "stage_blocks": [d, host_k, host_v, host_k.shape[0], t["table"], t["ctx"], t["sel"], t["cnt"], t["scores"], K,
                         t["smap"], t["stamp"], 1, K, True, t["pool_k"], t["pool_v"], t["moved"]],
        "sparse_decode_attn": [d, t["q"], T, t["pool_k"], t["pool_v"], t["smap"], K, t["ctx"], 0.5, t["out"], t["lse"],
                               t["ws"]],
    }


@pytest.mark.gpu
@pytest.mark.parametrize("tier", ["device", "pinned"])
def test_plain_calls_are_accepted(tier):
    """Every function takes the plain call itself (status 0, not None, which would be the Python binding's turn),
    on the current stream and on a handle, and leaves what the Python binding leaves."""
    L.lib()
    side = torch.cuda.Stream()
    outs = []
    for stream in ("python", None, side.cuda_stream):
        t = _tensors("cuda")
        host = [t[n] if tier == "device" else t[n].cpu().pin_memory() for n in ("host_k", "host_v")]
        torch.cuda.synchronize()
        keep = L._fast
        L._fast = None if stream == "python" else keep
        try:
            for name, args in _calls(t, *host).items():
                if stream == "python":
                    getattr(P, "oasis_" + name)(t["d"], *(args[1:3] + args[4:] if name == "stage_blocks" else args[1:]))
                else:
                    assert getattr(keep, name)(*args, stream) == 0, name
        finally:
            L._fast = keep
        torch.cuda.synchronize()
        outs.append([t[n].clone() for n in ("scores", "sel", "cnt", "smap", "stamp", "pool_k", "pool_v", "moved",
                                            "out", "lse")])
    for other in outs[1:]:
        assert all(torch.equal(x, y) for x, y in zip(outs[0], other))


@pytest.mark.gpu
def test_bad_counts_keep_the_bindings_errors():
    """Negative and overflowing counts match no tensor: the Python binding refuses them as it always did, before
    the library is called (in the native functions a negative product used to mean any count)."""
    L.lib()
    t = _tensors("cuda")
    host = t["host_k"], t["host_v"]
    at = {"score_blocks": (2,), "select_topk": (3,), "score_select": (2, 8), "stage_blocks": (3, 9),
          "sparse_decode_attn": (2, 6)}
    for name, places in at.items():
        for i in places:
            for bad in (-1, -2, -(1 << 31), (1 << 31) - 1):
                args = _calls(t, *host)[name]
                args[i] = bad
                assert getattr(L._fast, name)(*args, None) is None, (name, i, bad)
    for bad in (-1, -2):
        with pytest.raises(ValueError, match="sel: "):
            P.oasis_select_topk(t["d"], t["scores"], t["ctx"], bad, t["sel"], t["cnt"])
        with pytest.raises(ValueError, match="q: "):
            P.oasis_score_blocks(t["d"], t["q"], bad, 1, 2, t["kmax"], t["kmin"], t["ctx"], t["scores"])
    # 2^30 requests of 2^30 heads and 16 tokens: 2^64 rows are not the 0 rows of an empty tensor
    huge = P.dims(1 << 30, 1 << 30, 1, 128, B, NB)
    empty = t["q"][:0]
    call = [ctypes.addressof(huge), empty, 16, empty, empty, t["sel"][:0], 0, t["ctx"], None, empty, None, t["ws"], None]
    assert L._fast.sparse_decode_attn(*call) is None
    none = P.dims(R, H * G, H, 0, B, NB)  # no head dimension: the default scale does not exist
    with pytest.raises(ZeroDivisionError):
        P.oasis_sparse_decode_attn(none, empty, T, empty, empty, t["smap"], K, t["ctx"], None, empty, None, t["ws"])


@pytest.mark.gpu
def test_capture_takes_the_current_stream():
    """A captured step replays on its own stream and gives the eager results, replay after replay."""
    t, ref = _tensors("cuda"), _tensors("cuda")
    _step(ref)
    _step(t)
    torch.cuda.synchronize()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g):
        _step(t)
    for _ in range(3):
        for n in ("scores", "sel", "cnt", "out", "lse"):
            t[n].zero_()
        torch.cuda.synchronize()
        g.replay()
        torch.cuda.synchronize()
        for n in ("scores", "sel", "cnt", "out", "lse", "smap", "pool_k"):
            assert torch.equal(t[n], ref[n]), n


@pytest.fixture
def fresh_binding():
    """The binding as before its first call; restored afterwards."""
    keep = L._lib, L._fast
    L._lib = L._fast = None
    yield
    L._lib, L._fast = keep


def _missing():
    raise ImportError("no module named _fastcall")


@pytest.mark.parametrize("load,reason", [
    (_missing, "no module named"),
    (lambda: types.SimpleNamespace(__file__="old.so", bind=None), "abi_version"),  # built before it had a version
    (lambda: types.SimpleNamespace(__file__="old.so", bind=None, abi_version=L.ABI_VERSION - 1), "ABI version"),
])
def test_binding_works_without_a_fitting_module(fresh_binding, monkeypatch, load, reason):
    """The library alone is enough: the calls take the Python binding, and loading says so once."""
    monkeypatch.setattr(L, "_load_fast", load)
    with pytest.warns(RuntimeWarning, match=reason):
        L.lib()
    assert L._fast is None and P.oasis_abi_version() == L.ABI_VERSION
    t = _tensors("cpu")
    with pytest.raises(ValueError, match="scores must be a device tensor"):
        P.oasis_select_topk(t["d"], t["scores"], t["ctx"], K, t["sel"], t["cnt"], 0)


def test_built_module_fits_the_library(fresh_binding, recwarn):
    L.lib()
    assert L._fast is not None and L._fast.abi_version == L.ABI_VERSION
    assert not [w for w in recwarn if "marshalling" in str(w.message)]


def test_library_is_built_without_a_host_compiler(monkeypatch, tmp_path):
    """What fails is the module alone; the library is in place and no older module stays beside it."""
    from paper_2608_08097_amd import build_lib as b
    monkeypatch.setattr(b, "LIB_PATH", str(tmp_path / "liboasis.so"))
    monkeypatch.setattr(b, "FASTCALL_PATH", str(tmp_path / "_fastcall.so"))
    monkeypatch.setattr(b, "BUILD_DIR", str(tmp_path / "objs"))
    (tmp_path / "_fastcall.so").write_text("older")
    monkeypatch.setenv("CXX", str(tmp_path / "no-such-compiler"))
    run = b._run

    def fake(cmd):  # hipcc's part stands in for itself
        if cmd[0] != b.hipcc():
            return run(cmd)
        open(cmd[cmd.index("-o") + 1], "w").close()
        return ""

    monkeypatch.setattr(b, "_run", fake)
    with pytest.warns(RuntimeWarning, match="native marshalling was not built"):
        assert b.build() == str(tmp_path / "liboasis.so")
    assert (tmp_path / "liboasis.so").exists() and not (tmp_path / "_fastcall.so").exists()


def test_module_has_no_thread_local_storage():
    """Loading a module with a TLS segment slows every thread_local access of the libraries loaded before it."""
    import struct
    import paper_2608_08097_amd._fastcall as fast
    with open(fast.__file__, "rb") as f:
        head = f.read(64)
        off, size, count = struct.unpack_from("<Q", head, 32)[0], *struct.unpack_from("<HH", head, 54)
        f.seek(off)
        types = [struct.unpack_from("<I", f.read(size))[0] for _ in range(count)]
    assert 1 in types and 7 not in types  # PT_LOAD, PT_TLS
