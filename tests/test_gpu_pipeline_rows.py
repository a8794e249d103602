"""Pipelined steps with many attention rows (two teams of waves per workgroup, planned for the CUs that staging
leaves): the native issuer against the same schedule issued call by call, and against the oracle."""
import numpy as np
import pytest
import torch

import paper_2608_08097_amd as P
from oracle import oasis_oracle as O
from paper_2608_08097_amd.path import DecodePath
from tests.gpu_util import assert_attn_close, assert_lse_close, host_bits, note

pytestmark = pytest.mark.gpu

STEPS, LAYERS = 6, 2


def _run(native, R, Hq, H, T, B, k, NB, seed):
    g = torch.Generator(device="cuda").manual_seed(seed)

    def randn(*s):
        return torch.randn(s, generator=g, device="cuda", dtype=torch.bfloat16)

    pages = NB
    dev_k, dev_v = randn(pages, H, B, 128), randn(pages, H, B, 128)
    host = []
    for t in (dev_k, dev_v):
        h = torch.empty(t.shape, dtype=t.dtype, pin_memory=True)
        h.copy_(t)
        host.append(h)
    table = torch.stack([torch.randperm(pages, generator=g, device="cuda")[:NB] for _ in range(R)]).to(torch.int32)
    ctx = torch.randint(NB * B // 2, NB * B - STEPS, (R,), generator=g, device="cuda", dtype=torch.int32)
    d = P.dims(R, Hq, H, 128, B, NB)
    path = DecodePath(d, T, k, *host, table, fetch_cap=max(1, k // 20), native=native)
    layers = [path.new_layer() for _ in range(LAYERS)]
    for st in layers:
        path.build_summaries(st, ctx, dev_k)
    qs = [[randn(R, T, Hq, 128) for _ in range(STEPS)] for _ in layers]
    for st, q in zip(layers, qs):  # the working set when decoding starts: the first prediction, uncapped
        path.predict(st, q[0], ctx)
        path.stage(st, ctx, 0, fetch_cap=k)
    torch.cuda.synchronize()
    before = []
    for t in range(STEPS):
        if t == STEPS - 1:
            torch.cuda.synchronize()
            before = [(st.pool_k[-1:].clone(), st.pool_v[-1:].clone(), st.slot_map[-1:].clone()) for st in layers]
        for st, q in zip(layers, qs):
            path.step_pipelined(st, q[t], ctx, t + 1)
    path.join()
    path.check()
    torch.cuda.synchronize()
    return path, layers, qs, ctx, before


# (requests, query heads, KV heads, tokens, B, k): 48 pairs of 35 rows, 4 splits instead of 5; 24 pairs at B = 32;
# 128 pairs of 72 rows, one split instead of two; 33 x 8 pairs of 64 rows, one team per pair
@pytest.mark.parametrize("R,Hq,H,T,B,k,NB", [(12, 20, 4, 7, 16, 128, 260), (3, 40, 8, 7, 32, 64, 140),
                                              (16, 64, 8, 9, 32, 60, 130), (33, 64, 8, 8, 16, 24, 60)])
def test_many_row_steps(R, Hq, H, T, B, k, NB):
    note(f"many-row pipelined steps R={R} Hq={Hq} H={H} T={T} B={B} k={k}")
    path, layers, qs, ctx, before = _run(True, R, Hq, H, T, B, k, NB, R + T)
    _, ref, _, _, _ = _run(False, R, Hq, H, T, B, k, NB, R + T)
    for l, (st, rf, (pk, pv, sm)) in enumerate(zip(layers, ref, before)):
        for name in ("scores", "sel", "sel_count", "slot_map", "slot_stamp", "pool_k", "pool_v", "moved"):
            assert torch.equal(getattr(st, name), getattr(rf, name)), (l, name)
        q = qs[l][STEPS - 1][-1:]
        o, lse = O.sparse_attend(host_bits(q), host_bits(pk), np.ascontiguousarray(np.swapaxes(host_bits(pv), -1, -2)),
                                 sm.cpu().numpy(), ctx[-1:].cpu().numpy(), B)
        for s in (st, rf):
            assert_attn_close(host_bits(s.out[-1:]), o)
            assert_lse_close(s.lse[-1:].cpu().numpy(), lse)
        # the two forms round the same sums in another order: bf16 outputs within two steps of the larger
        a, b = st.out.float(), rf.out.float()
        assert torch.all((a - b).abs() <= 2.0 ** -7 * torch.maximum(a.abs(), b.abs()) + 2e-3)
        assert torch.allclose(st.lse, rf.lse, rtol=1e-5, atol=1e-4)
