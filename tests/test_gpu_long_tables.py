"""Tables sized for long contexts holding short ones: the work a call does follows the contexts, and the results
are those of tables that just fit."""
import numpy as np
import pytest
import torch

import paper_2608_08097_amd as P
from tests.gpu_util import note

pytestmark = pytest.mark.gpu

B, D = 16, 128


def _inputs(seed, R, H, Hq, T, NB, n_cand):
    g = torch.Generator(device="cuda").manual_seed(seed)
    a = torch.randn((R, H, NB, D), generator=g, device="cuda", dtype=torch.bfloat16)
    b = torch.randn((R, H, NB, D), generator=g, device="cuda", dtype=torch.bfloat16)
    ctx = torch.tensor([B * n + 1 + 5 * (n % 3) if n else 7 for n in n_cand], dtype=torch.int32, device="cuda")
    return torch.randn((R, T, Hq, D), generator=g, device="cuda", dtype=torch.bfloat16), torch.maximum(a, b), \
        torch.minimum(a, b), ctx


def _scores(q, kmax, kmin, ctx):
    R, H, NB, _ = kmax.shape
    T = q.shape[1]
    s = torch.full((R, H, NB), 7.0, device="cuda")
    P.oasis_score_blocks(P.dims(R, q.shape[2], H, D, B, NB), q, T, 1, T - 1, kmax, kmin, ctx, s)
    return s


# 1 to 4 row tiles; candidates at the edges of a wave's tiles and of a workgroup's 128 or 256 blocks
@pytest.mark.parametrize("Hq,T", [(32, 5), (64, 5), (40, 9), (64, 9)])
def test_scores_do_not_depend_on_the_table_length(Hq, T):
    n_cand = [0, 1, 31, 64, 127, 128, 129, 255, 256, 257, 300, 383, 384]
    H, NB, long = 8, 385, 3000
    q, kmax, kmin, ctx = _inputs(Hq + T, len(n_cand), H, Hq, T, NB, n_cand)
    note(f"scores in long tables Hq={Hq} T={T}")
    ref = _scores(q, kmax, kmin, ctx)
    pad = [torch.full((len(n_cand), H, long, D), float("nan"), dtype=torch.bfloat16, device="cuda") for _ in range(2)]
    pad[0][:, :, :NB], pad[1][:, :, :NB] = kmax, kmin
    got = _scores(q, *pad, ctx)
    torch.cuda.synchronize()
    assert torch.equal(got[:, :, :NB], ref) and torch.all(got[:, :, NB:] == -float("inf"))
    for i, n in enumerate(n_cand):
        assert torch.all(ref[i, :, n:] == -float("inf")) and torch.all(torch.isfinite(ref[i, :, :n]))
        rows = q[i, 1:].double().view(T - 1, H, Hq // H, D)
        for h in (0, H - 1):
            x = rows[:, h].reshape(-1, 1, D)
            want = torch.maximum(x * kmax[i, h, :n].double(), x * kmin[i, h, :n].double()).sum(-1).amax(0)
            # fp32 sums of 256 exact products
            assert torch.all((ref[i, h, :n].double() - want).abs() <= 1e-3 + 1e-5 * want.abs())


def _time_us(call, n=40):
    call()
    torch.cuda.synchronize()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g):
        for _ in range(n):
            call()
    times = []
    for _ in range(7):
        a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        a.record()
        g.replay()
        b.record()
        torch.cuda.synchronize()
        times.append(1000.0 * a.elapsed_time(b) / n)
    return sorted(times)[3]


@pytest.mark.parametrize("Hq,T", [(32, 5), (64, 5), (64, 9)])
def test_short_contexts_in_long_tables_cost_little_more(Hq, T):
    """Both sides score the same blocks; the long table adds its padding (4 MB of scores). Measured: 16 rows 6.6
    against 11.9 us, 32 rows 7.0 and 13.2, 64 rows 7.6 and 14.5 (1.8 to 1.9 times); with every workgroup of the
    table reading and multiplying, 24.1, 28.3 and 34.3 (3.7 to 4.5 times). The bound lies between."""
    R, H, NB, long = 16, 8, 500, 8000
    q, kmax, kmin, ctx = _inputs(3, R, H, Hq, T, NB, [250 + 15 * i for i in range(R)])
    pad = [torch.zeros((R, H, long, D), dtype=torch.bfloat16, device="cuda") for _ in range(2)]
    pad[0][:, :, :NB], pad[1][:, :, :NB] = kmax, kmin
    note(f"time of scores in long tables Hq={Hq} T={T}")
    out = {}
    for name, (mx, mn) in (("fit", (kmax, kmin)), ("long", pad)):
        n = mx.shape[2]
        s, d = torch.empty((R, H, n), device="cuda"), P.dims(R, Hq, H, D, B, n)
        out[name] = _time_us(lambda: P.oasis_score_blocks(d, q, T, 1, T - 1, mx, mn, ctx, s))
    note(f"scores: fitting table {out['fit']:.1f} us, long table {out['long']:.1f} us")
    assert out["long"] <= 2.7 * out["fit"]


def _summaries(pages, table, ctx, NB, block):
    R, H = table.shape[0], pages.shape[1]
    out = [torch.zeros((R, H, NB, D), dtype=torch.bfloat16, device="cuda") for _ in range(2)]
    d = P.dims(R, H, H, D, block, NB)
    return out, lambda: P.oasis_build_summaries(d, pages, table, ctx, *out)


# the plain form alone, and one request long enough for the non-temporal form beside short ones
@pytest.mark.parametrize("block,n_cand", [(16, [0, 1, 40, 300]), (32, [5, 0, 150]), (16, [2100, 3, 700, 0]),
                                          (32, [1100, 2, 333])])
def test_summaries_do_not_depend_on_the_table_length(block, n_cand):
    R, H, long = len(n_cand), 8, 4000
    g = torch.Generator(device="cuda").manual_seed(block + R)
    NB = max(n_cand) + 1
    pages = torch.randn((R * NB, H, block, D), generator=g, device="cuda", dtype=torch.bfloat16)
    perm = torch.randperm(R * NB, generator=g, device="cuda").to(torch.int32).view(R, NB)
    ctx = torch.tensor([block * n + 1 for n in n_cand], dtype=torch.int32, device="cuda")
    for nb in (NB, long):
        table = torch.full((R, nb), -1, dtype=torch.int32, device="cuda")
        table[:, :NB] = perm
        note(f"summaries B={block} candidates={n_cand} table={nb}")
        (kmax, kmin), call = _summaries(pages, table, ctx, nb, block)
        call()
        torch.cuda.synchronize()
        for r, n in enumerate(n_cand):
            keys = pages[perm[r, :n].long()]
            for got, ext in ((kmax, keys.amax(2) if n else None), (kmin, keys.amin(2) if n else None)):
                assert not got[r, :, n:].any()
                assert n == 0 or torch.equal(got[r, :, :n], ext.transpose(0, 1))


def test_short_summaries_in_long_tables_cost_little_more():
    """75 MB of keys, found in the cache: the table's length adds workgroups that end at once, and does not change
    how the keys are read. Measured: 14.5 against 15.6 us (1.06 to 1.08 times); read past the caches 19.3 (1.34)."""
    block = 32
    R, H, tokens, long = 16, 8, 2304, 96000 // block
    n = tokens // block
    pages = torch.randn((R * n, H, block, D), device="cuda", dtype=torch.bfloat16)
    ctx = torch.full((R,), tokens - 3, dtype=torch.int32, device="cuda")
    out = {}
    for name, nb in (("fit", n), ("long", long)):
        table = torch.full((R, nb), -1, dtype=torch.int32, device="cuda")
        table[:, :n] = torch.arange(R * n, dtype=torch.int32, device="cuda").view(R, n)
        note(f"time of summaries B={block} table={nb}")
        out[name] = _time_us(_summaries(pages, table, ctx, nb, block)[1])
    note(f"summaries: fitting table {out['fit']:.1f} us, long table {out['long']:.1f} us")
    assert out["long"] <= 1.2 * out["fit"]
