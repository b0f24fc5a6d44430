"""Row operators on rows of any length, pitch and start, which the register kernels take as overlapping chunks: lengths at
the edges of a chunk and of every (threads, chunks) pair, against the oracle with the bounds of test_gpu_memops.py."""
import numpy as np
import pytest

from tests.helpers import dev
from tests.test_gpu_memops import _check, _gen, _host, _out, _pitched

pytestmark = pytest.mark.gpu

SHAPES = [  # rows, cols, pitch padding, elements the buffers start past an aligned address
    (5, 3, 0, 0), (6, 9, 0, 1), (7, 15, 2, 0), (3, 513, 1, 3), (33, 791, 0, 0), (4, 1025, 0, 1), (5, 2055, 3, 0), (3, 4097, 0, 2),
    (2, 8193, 1, 0), (2, 16385, 0, 1), (2, 32771, 0, 0), (1, 65537, 0, 0), (3, 1000, 0, 1),
]


@pytest.mark.parametrize("op", ["softmax", "layernorm", "rmsnorm"])
@pytest.mark.parametrize("kinds", [("f32", "f32"), ("bf16", "f32"), ("bf16", "bf16"), ("f32", "bf16")])
def test_rows_of_any_length(op, kinds, oracle):
    from paper_2505_02146_amd import xp
    kin, kout = kinds
    for rows, cols, pad, skew in SHAPES:
        x = _gen(kin, (rows, cols), 1, sigma=2.0)
        g, b = _gen(kin, (cols,), 2), _gen(kin, (cols,), 3)
        ld = cols + pad
        xb = _pitched(x, ld, 0x7FC0 if kin == "bf16" else np.nan)           # NaNs between the rows must not count
        shifted = lambda a: dev(np.concatenate([a[:1].repeat(skew), a]))[skew:]
        y = _out(kout, skew + rows * ld, -3.0)
        if op == "softmax":
            xp.xp_softmax(rows, cols, shifted(xb), ld, y[skew:], ld, x_type=kin)
            ref = oracle.softmax(xb, rows=rows, cols=cols, ldx=ld)
        elif op == "layernorm":
            xp.xp_layernorm(rows, cols, shifted(xb), ld, shifted(g), shifted(b), 1e-5, y[skew:], ld, x_type=kin)
            ref = oracle.layernorm(xb, rows=rows, cols=cols, gamma=g, beta=b, eps=1e-5, ldx=ld)
        else:
            xp.xp_rmsnorm(rows, cols, shifted(xb), ld, shifted(g), 1e-6, y[skew:], ld, x_type=kin)
            ref = oracle.rmsnorm(xb, rows=rows, cols=cols, gamma=g, eps=1e-6, ldx=ld)
        got = _host(y)[skew:].reshape(rows, ld)
        _check(np.ascontiguousarray(got[:, :cols]), ref, f"{op} {kinds} {(rows, cols, pad, skew)}")
        assert (got[:, cols:] == (0xC040 if kout == "bf16" else -3.0)).all(), "wrote between the rows"


@pytest.mark.parametrize("cols", [201, 3001])
def test_odd_rows_in_place(cols, oracle):
    from paper_2505_02146_amd import xp
    x = _gen("bf16", (17, cols), 5)
    buf = dev(x.reshape(-1))
    xp.xp_softmax(17, cols, buf, cols, buf, cols, x_type="bf16", y_type="bf16")
    _check(buf.cpu().numpy().view(np.uint16).reshape(17, cols), oracle.softmax(x.reshape(-1), rows=17, cols=cols), "in place")
