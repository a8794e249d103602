"""Attention over the ways a call is cut up: pair counts around the workgroup and XCD boundaries, splits long
enough for several slot-map chunks per wave, and slot maps whose free slots come in runs (units that are never
read), against the oracle at the attention tolerance."""
import numpy as np
import pytest
import torch

import paper_2608_08097_amd as P
from oracle import oasis_oracle as O
from tests.gpu_util import (assert_attn_close, assert_lse_close, dev_bf16, dev_i32, host_bits, note,
                            pool_v_from_htd)
from workloads import random_bf16

pytestmark = pytest.mark.gpu

CASES = [
    # (seed, R, Hq, Hkv, T, B, k_slots, free slots)
    (1, 1, 4, 1, 5, 16, 4300, "tail"),       # 34 units per wave: a second slot-map chunk, none of it attended
    (2, 1, 4, 1, 5, 16, 4300, "islands"),    # a few attended slots far apart
    (3, 1, 4, 1, 5, 16, 4301, "head"),       # the first chunk free, an odd slot count
    (4, 1, 2, 1, 4, 32, 4225, "islands"),    # B = 32: 64 units per chunk, one row tile
    (5, 1, 8, 1, 9, 16, 1400, "islands"),    # many-row kernel over several chunks per split
    (6, 1, 8, 1, 7, 32, 1700, "tail"),
    (7, 5, 8, 2, 5, 16, 40, "tail"),         # 10 pairs: XCDs of two pairs and of one
    (8, 3, 1, 1, 3, 16, 60, "random"),       # 3 pairs, fewer than XCDs
    (9, 9, 5, 1, 2, 32, 30, "random"),       # 9 pairs
    (10, 17, 16, 8, 9, 16, 24, "random"),    # 136 pairs: two splits would need a second round of workgroups
    (11, 17, 64, 8, 9, 16, 25, "tail"),      # the same with five row tiles, an odd unit count
    (12, 5, 32, 8, 8, 32, 33, "random"),     # 40 pairs x 32 rows: six splits, not seven
    (13, 33, 16, 8, 5, 16, 16, "tail"),      # 264 pairs: more than CUs
    (14, 43, 24, 6, 9, 16, 12, "random"),    # 258 pairs x 36 rows: many-row kernel, one team per pair
    (15, 65, 64, 8, 7, 32, 5, "random"),     # 520 pairs x 56 rows: more than two per CU
    (16, 1, 16, 1, 3, 16, 130, "random"),    # 48 rows, 66 units: many short splits
    (17, 33, 56, 8, 7, 16, 9, "random"),     # one team per pair: four row tiles (49 rows), 264 pairs
    (18, 43, 48, 6, 8, 32, 4, "tail"),       # the same at B = 32, 64 rows, 258 pairs
    (19, 33, 40, 8, 7, 32, 6, "random"),     # three row tiles at B = 32
    (20, 257, 2, 1, 17, 16, 66, "islands"),  # 34 units per split: a second slot-map chunk
]


def _slots(rng, kind, shape):
    ids = rng.integers(0, 10 ** 6, shape).astype(np.int32)
    ks = shape[-1]
    at = np.arange(ks)
    if kind == "random":
        free = rng.random(shape) < 0.3
    elif kind == "tail":  # a context shorter than the budget: a random number of leading slots is filled
        free = at >= rng.integers(0, max(1, ks // 3), shape[:-1])[..., None]
    elif kind == "head":
        free = np.broadcast_to(at < ks - ks // 8, shape)
    else:
        free = rng.random(shape) >= 4.0 / ks
    return np.where(free, np.int32(-1), ids)


@pytest.mark.parametrize("seed,R,Hq,Hkv,T,B,ks,kind", CASES)
def test_attn_splits(seed, R, Hq, Hkv, T, B, ks, kind):
    rng = np.random.default_rng(1700 + seed)
    q = random_bf16(1710 + seed, (R, T, Hq, 128))
    pk = random_bf16(1720 + seed, (R, ks + 1, Hkv, B, 128))
    pv = random_bf16(1730 + seed, (R, ks + 1, Hkv, B, 128))
    smap = _slots(rng, kind, (R, Hkv, ks))
    ctx = rng.integers(0, (ks + 2) * B, R).astype(np.int32)
    free = np.swapaxes(smap < 0, 1, 2)  # [R][ks][Hkv]
    pk[:, :ks][free] = np.uint16(0x7FC0)  # NaN in every free slot must not leak
    pv[:, :ks][free] = np.uint16(0x7FC0)
    ref_o, ref_l = O.sparse_attend(q, pk, pv, smap, ctx, B)
    note(f"attn splits seed={seed} R={R} Hq={Hq} Hkv={Hkv} T={T} B={B} ks={ks} {kind}")
    d = P.dims(R, Hq, Hkv, 128, B, ks + 2)
    out = torch.full((R, T, Hq, 128), float("nan"), dtype=torch.bfloat16, device="cuda")
    lse = torch.full((R, T, Hq), float("nan"), dtype=torch.float32, device="cuda")
    ws = torch.zeros(P.oasis_attn_workspace_bytes(d, T, ks), dtype=torch.uint8, device="cuda")
    args = (d, dev_bf16(q), T, dev_bf16(pk), dev_bf16(pool_v_from_htd(pv)), dev_i32(smap), ks, dev_i32(ctx), None)
    for _ in range(2):
        P.oasis_sparse_decode_attn(*args, out, lse, ws)
    torch.cuda.synchronize()
    assert_attn_close(host_bits(out), ref_o)
    assert_lse_close(lse.cpu().numpy(), ref_l)


@pytest.mark.parametrize("R,Hq,T,B,ks", [(13, 32, 5, 16, 128), (25, 32, 1, 32, 64), (32, 64, 5, 32, 64)])
def test_attn_past_the_caches(R, Hq, T, B, ks):
    """Calls over 96 MB take the non-temporal loads (both split kernels; B = 32 with the CUs full for the many-row
    one), against the oracle on the first and the last request."""
    Hkv = 8
    g = torch.Generator(device="cuda").manual_seed(R)
    shape = (R, ks + 1, Hkv, B, 128)
    pk = torch.randn(shape, generator=g, device="cuda", dtype=torch.bfloat16)
    pv = torch.randn((R, ks + 1, Hkv, 128, B), generator=g, device="cuda", dtype=torch.bfloat16)
    q = torch.randn((R, T, Hq, 128), generator=g, device="cuda", dtype=torch.bfloat16)
    smap = torch.arange(ks, dtype=torch.int32, device="cuda").expand(R, Hkv, ks).contiguous()
    ctx = torch.full((R,), (ks + 1) * B - 3, dtype=torch.int32, device="cuda")
    assert pk.numel() * 4 > 96 << 20
    d = P.dims(R, Hq, Hkv, 128, B, ks + 2)
    out, lse = torch.empty_like(q), torch.empty((R, T, Hq), device="cuda")
    ws = torch.zeros(max(1, P.oasis_attn_workspace_bytes(d, T, ks)), dtype=torch.uint8, device="cuda")
    note(f"attn past the caches R={R} Hq={Hq} T={T} B={B} ks={ks}")
    P.oasis_sparse_decode_attn(d, q, T, pk, pv, smap, ks, ctx, None, out, lse, ws)
    torch.cuda.synchronize()
    for r in (0, R - 1):
        bits = [host_bits(x[r:r + 1]) for x in (q, pk, pv)]
        ref_o, ref_l = O.sparse_attend(bits[0], bits[1], np.ascontiguousarray(np.swapaxes(bits[2], -1, -2)),
                                       smap[r:r + 1].cpu().numpy(), ctx[r:r + 1].cpu().numpy(), B)
        assert_attn_close(host_bits(out[r:r + 1]), ref_o)
        assert_lse_close(lse[r:r + 1].cpu().numpy(), ref_l)


@pytest.mark.parametrize("R,Hq,T,B,ks", [(25, 32, 2, 16, 128), (16, 64, 9, 32, 128), (25, 32, 5, 32, 64)])
def test_attn_past_the_caches_with_free_slots(R, Hq, T, B, ks):
    """The same forms at one row tile (B = 16), five and two (B = 32), with single free slots, runs of them (units
    that are never read) and NaN in all of them; first, middle and last request."""
    Hkv = 8
    g = torch.Generator(device="cuda").manual_seed(R + T)
    pk = torch.randn((R, ks + 1, Hkv, B, 128), generator=g, device="cuda", dtype=torch.bfloat16)
    pv = torch.randn((R, ks + 1, Hkv, 128, B), generator=g, device="cuda", dtype=torch.bfloat16)
    q = torch.randn((R, T, Hq, 128), generator=g, device="cuda", dtype=torch.bfloat16)
    at = torch.arange(ks, device="cuda")
    start = torch.randint(0, ks, (R, Hkv, 1), generator=g, device="cuda")
    free = (torch.rand((R, Hkv, ks), generator=g, device="cuda") < 0.2) | ((at >= start) & (at < start + ks // 4))
    smap = torch.where(free, -1, at.expand(R, Hkv, ks)).to(torch.int32).contiguous()
    for pool in (pk, pv):
        pool[:, :ks][free.transpose(1, 2)] = float("nan")
    ctx = torch.randint((ks + 1) * B - B + 1, (ks + 1) * B + 1, (R,), generator=g, device="cuda", dtype=torch.int32)
    assert pk.numel() * 4 > 96 << 20
    d = P.dims(R, Hq, Hkv, 128, B, ks + 2)
    out, lse = torch.empty_like(q), torch.empty((R, T, Hq), device="cuda")
    ws = torch.zeros(max(1, P.oasis_attn_workspace_bytes(d, T, ks)), dtype=torch.uint8, device="cuda")
    note(f"attn past the caches, free slots R={R} Hq={Hq} T={T} B={B} ks={ks}")
    P.oasis_sparse_decode_attn(d, q, T, pk, pv, smap, ks, ctx, None, out, lse, ws)
    torch.cuda.synchronize()
    for r in (0, R // 2, R - 1):
        bits = [host_bits(x[r:r + 1]) for x in (q, pk, pv)]
        ref_o, ref_l = O.sparse_attend(bits[0], bits[1], np.ascontiguousarray(np.swapaxes(bits[2], -1, -2)),
                                       smap[r:r + 1].cpu().numpy(), ctx[r:r + 1].cpu().numpy(), B)
        assert_attn_close(host_bits(out[r:r + 1]), ref_o)
        assert_lse_close(lse[r:r + 1].cpu().numpy(), ref_l)


def test_summaries_and_scores_past_the_caches():
    """The non-temporal forms of the summaries (from 192 MB of keys) and of the vector-ALU scorer (from 96 MB)
    against torch's extrema (exact) and the 64-bit bound (fp32 sums: 1e-5 of the score, 1e-3)."""
    R, H, NB, B = 7, 8, 7000, 16
    g = torch.Generator(device="cuda").manual_seed(5)
    pages = torch.randn((R * NB, H, B, 128), generator=g, device="cuda", dtype=torch.bfloat16)
    table = torch.randperm(R * NB, generator=g, device="cuda").to(torch.int32).view(R, NB).contiguous()
    ctx = torch.tensor([NB * B - 5 - 1000 * r for r in range(R)], dtype=torch.int32, device="cuda")
    kmax = torch.zeros((R, H, NB, 128), dtype=torch.bfloat16, device="cuda")
    kmin = torch.zeros_like(kmax)
    d = P.dims(R, H, H, 128, B, NB)
    q = torch.randn((R, 2, H, 128), generator=g, device="cuda", dtype=torch.bfloat16)
    scores = torch.empty((R, H, NB), device="cuda")
    note("summaries and scores past the caches")
    P.oasis_build_summaries(d, pages, table, ctx, kmax, kmin)
    P.oasis_score_blocks(d, q, 2, 1, 1, kmax, kmin, ctx, scores)
    torch.cuda.synchronize()
    for r in (0, 3, R - 1):
        nc = (int(ctx[r]) + B - 1) // B - 1
        keys = pages[table[r, :nc].long()]
        for got, want in ((kmax, keys.amax(2)), (kmin, keys.amin(2))):
            assert torch.equal(got[r, :, :nc], want.transpose(0, 1)) and not got[r, :, nc:].any()
        qd = q[r, 1].double()[:, None, :]
        ref = torch.maximum(qd * kmax[r, :, :nc].double(), qd * kmin[r, :, :nc].double()).sum(-1)
        assert torch.all((scores[r, :, :nc].double() - ref).abs() <= 1e-3 + 1e-5 * ref.abs())
        assert torch.all(scores[r, :, nc:] == -float("inf"))
