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
