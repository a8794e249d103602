"""Top-K over the ways a row is selected: every key count per thread, wanted bins small enough to be ranked
directly and too full for it (or ranked at 64 keys exactly), ties at the cut that span waves and rounds, and
rows whose keys are re-read from memory. Selections are exact: compared with the oracle id for id. The fused
score + select kernel must give the two kernels' selections on the same rows."""
import numpy as np
import pytest
import torch

import paper_2608_08097_amd as P
from oracle import oasis_oracle as O
from tests.gpu_util import dev_bf16, dev_i32, note
from workloads import random_bf16

pytestmark = pytest.mark.gpu

CASES = [
    # (seed, R, H, NBmax, candidates per request, k, scores)
    (1, 2, 2, 70, [69, 66], 65, "normal"),             # a few candidates more than k
    (2, 3, 1, 2048, [2047, 513, 512], 128, "normal"),  # 512 threads, four keys each; edges of a round
    (3, 3, 1, 2049, [2048, 1025, 1024], 128, "ties"),  # 1,024 threads; edges of a round
    (4, 2, 2, 8192, [8191, 4000], 256, "outliers"),    # most keys in the lowest bins, a few far above
    (5, 2, 1, 8200, [8199, 8193], 128, "equal"),       # every score equal: an empty key range
    (6, 1, 2, 12000, [11999], 1000, "bin64"),          # exactly 64 keys in the wanted bin
    (7, 1, 2, 12000, [11999], 1000, "bin65"),          # one more: the passes go on
    (8, 1, 1, 33000, [32999], 512, "ties"),            # keys re-read from memory, ties across chunks of 32 rounds
    (9, 1, 1, 70000, [69999], 4000, "normal"),
    (10, 2, 1, 40000, [39999, 100], 65536, "ties"),    # k above the candidates
    (11, 1, 2, 3000, [2999], 128, "extreme"),          # the whole exponent range, both signs
]


def _scores(rng, kind, shape, n):
    if kind == "normal":
        s = rng.standard_normal(shape) * 50
    elif kind == "ties":
        s = rng.integers(-3, 4, shape) * 1.0
    elif kind == "outliers":
        s = rng.standard_normal(shape) * 1e-3
        s[..., rng.permutation(n)[:40]] += 1000.0
    elif kind == "equal":
        s = np.full(shape, -2.5)
    elif kind == "extreme":
        s = rng.choice([-1.0, 1.0], shape) * np.exp2(rng.uniform(-120, 120, shape))
    else:
        # 0 .. 255 in steps of 1 (a bin each), 999 of them above 128; the bin of 128 holds `m` close values
        m = int(kind[3:])
        s = rng.integers(0, 128, shape).astype(np.float64)
        ids = rng.permutation(n)
        s[..., ids[:990]] = rng.integers(129, 256, 990)
        s[..., ids[990:990 + m]] = 128.0 + rng.permutation(m) / 1024.0
        s[..., ids[990 + m]] = 255.0
        s[..., ids[990 + m + 1]] = 0.0
    return s.astype(np.float32)


@pytest.mark.parametrize("seed,R,H,NB,ncand,k,kind", CASES)
def test_select_paths(seed, R, H, NB, ncand, k, kind):
    rng = np.random.default_rng(2600 + seed)
    scores = _scores(rng, kind, (R, H, NB), max(ncand))
    ctx = np.array([16 * (n + 1) for n in ncand], np.int32)
    ref_sel, ref_cnt = O.select_topk(scores, ctx, k, 16)
    note(f"select paths seed={seed} NB={NB} k={k} {kind}")
    d = P.dims(R, H, H, 128, 16, NB)
    sel = torch.full((R, H, k), -7, dtype=torch.int32, device="cuda")
    cnt = torch.full((R, H), -7, dtype=torch.int32, device="cuda")
    P.oasis_select_topk(d, torch.from_numpy(scores).cuda(), dev_i32(ctx), k, sel, cnt)
    torch.cuda.synchronize()
    assert np.array_equal(cnt.cpu().numpy(), ref_cnt)
    assert np.array_equal(sel.cpu().numpy(), ref_sel)


# (seed, requests, rows per KV head, NBmax, candidates, k): rounds of 256 blocks per workgroup, keys per thread 4 to 32
FUSED = [(1, 3, 8, 2048, [2047, 257, 255], 128), (2, 2, 32, 2050, [2049, 16], 64), (3, 1, 17, 8190, [8189], 100),
         (4, 1, 5, 16384, [16383], 300), (5, 3, 20, 300, [0, 1, 299], 128)]


@pytest.mark.parametrize("seed,R,rows,NB,ncand,k", FUSED)
def test_score_select_paths(seed, R, rows, NB, ncand, k):
    """One KV head, `rows` query heads and one draft token."""
    q = random_bf16(2700 + seed, (R, 2, rows, 128))
    x = random_bf16(2710 + seed, (R, 1, NB, 128))
    y = random_bf16(2720 + seed, (R, 1, NB, 128))
    vx, vy = O.bf16_to_f64(x), O.bf16_to_f64(y)
    ctx = np.array([16 * (n + 1) if n else 5 for n in ncand], np.int32)
    d = P.dims(R, rows, 1, 128, 16, NB)
    args = (dev_bf16(q), 2, 1, 1, dev_bf16(np.where(vx >= vy, x, y)), dev_bf16(np.where(vx >= vy, y, x)), dev_i32(ctx))
    got = []
    for fused in (False, True):
        s = torch.full((R, 1, NB), 7.0, device="cuda")
        sel = torch.full((R, 1, k), -7, dtype=torch.int32, device="cuda")
        cnt = torch.full((R, 1), -7, dtype=torch.int32, device="cuda")
        note(f"score + select rows={rows} NB={NB} fused={fused}")
        if fused:
            P.oasis_score_select(d, *args, k, s, sel, cnt)
        else:
            P.oasis_score_blocks(d, *args, s)
            P.oasis_select_topk(d, s, args[-1], k, sel, cnt)
        torch.cuda.synchronize()
        got.append([t.cpu().numpy() for t in (s, sel, cnt)])
    for a, b in zip(*got):
        assert np.array_equal(a, b)
    ref_sel, ref_cnt = O.select_topk(got[0][0], ctx, k, 16)  # on the kernel's own fp32 scores: exact
    assert np.array_equal(got[0][1], ref_sel) and np.array_equal(got[0][2], ref_cnt)
