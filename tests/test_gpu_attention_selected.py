"""Attention as selection runs it where many workgroups are needed: the eight-wave kernels and, over many keys, the one with two
query blocks per wave, with ragged queries, ragged keys and padded pitches, a few problems of each call against the oracle
(gates and bound of test_gpu_attention.py)."""
import numpy as np
import pytest

from tests.test_gpu_attention import TIGHT, _gate, xp  # noqa: F401

pytestmark = pytest.mark.gpu

CASES = [  # batch, Lq, Lk, d, variant
    (256, 200, 257, 64, 5),                              # 512 workgroups of 128 queries
    (171, 300, 191, 64, 5),                              # 513: a second round of one is no round, see below
    (128, 200, 257, 128, 6),                             # 256 workgroups of 128 queries
    (130, 130, 64, 128, 6),
    (256, 200, 2049, 128, 6),                            # 256 of 256 queries, over many keys
    (116, 399, 2111, 128, 6),                            # 232
    (64, 1024, 2048, 128, 6),                            # whole tiles
]


@pytest.mark.parametrize("case", CASES)
@pytest.mark.parametrize("scale", [0.1, -0.15])
def test_selected_kernel_on_ragged_calls(xp, oracle, case, scale):  # noqa: F811
    import torch
    batch, Lq, Lk, d, variant = case
    if case == CASES[1]:
        variant = 2                                      # the four-wave kernel
    g = torch.Generator(device="cuda").manual_seed(3)
    ld = [d + 8, d + 16, d + 24, d + 4]                  # pitches of Q, K, V, O
    rows = [Lq, Lk, Lk, Lq]
    st = [r * l + 8 for r, l in zip(rows, ld)]           # batch strides, a gap behind each slice
    bufs = []
    for i in range(3):                                   # NaN wherever a row or slice does not reach
        t = torch.full((batch * st[i],), float("nan"), device="cuda", dtype=torch.bfloat16)
        view = t.view(batch, st[i])[:, :rows[i] * ld[i]].view(batch, rows[i], ld[i])
        view[:, :, :d] = torch.randn(batch, rows[i], d, device="cuda", generator=g).bfloat16()
        bufs.append(t)
    o = torch.full((batch * st[3],), -7.0, device="cuda")
    xp.xp_force_config(xp.XP_OP_ATTENTION, "bf16", -1)
    xp.xp_attention(batch, Lq, Lk, d, d, scale, bufs[0], ld[0], st[0], bufs[1], ld[1], st[1], bufs[2], ld[2], st[2], o, ld[3], st[3])
    assert xp.xp_last_config(xp.XP_OP_ATTENTION, "bf16") == variant
    out = o.view(batch, st[3])[:, :Lq * ld[3]].view(batch, Lq, ld[3])
    assert (out[:, :, d:] == -7.0).all() and (o.view(batch, st[3])[:, Lq * ld[3]:] == -7.0).all(), "wrote outside the output"
    assert torch.isfinite(out[:, :, :d]).all()
    for b in (0, batch // 2, batch - 1):
        q, k, v = (t[b * s:b * s + r * l].view(torch.int16).cpu().numpy().view(np.uint16) for t, s, r, l in zip(bufs, st, rows, ld))
        ref = oracle.attention(q, k, v, batch=1, Lq=Lq, Lk=Lk, d=d, dv=d, scale=scale, ldq=ld[0], ldk=ld[1], ldv=ld[2])
        _gate(out[b:b + 1, :, :d].cpu().numpy(), ref, f"{case} scale {scale} problem {b}", TIGHT[variant])
