"""The convolution kernel for few input channels, forced at the edges of its runs, steps and tiles, against the oracle."""
import numpy as np
import pytest

from paper_2505_02146_amd import inputs
from tests.helpers import check_float, dev

pytestmark = pytest.mark.gpu

NAN_BITS = 0x7FC0


@pytest.fixture(scope="module")
def xp():
    from paper_2505_02146_amd import xp as m
    yield m
    for op in (0, 1, 2):
        for t in ("bf16", "i8"):
            m.xp_force_config(op, t, -1)


def _variant(xp, op, kind, text):
    found = [v for v in range(xp.xp_num_configs(op, kind)) if text in xp.xp_describe_config(op, kind, v)]
    assert len(found) == 1
    return found[0]


CONVS = [
    # N, H, W, Cin, Cout, R, S, stride, pad
    (2, 30, 37, 3, 64, 7, 7, (2, 2), (3, 3)),           # even distance of pixels; a row of 19 outputs, two groups
    (2, 21, 33, 3, 70, 3, 3, (1, 1), (1, 1)),           # odd distance; a second block of channels, its edge inside four
    (1, 8, 9, 1, 5, 3, 3, (1, 1), (1, 1)),              # one chunk a run; fewer channels than a block
    (3, 17, 260, 4, 32, 5, 5, (1, 2), (2, 2)),          # several parts or rows a tile
    (1, 40, 600, 4, 16, 7, 7, (1, 1), (3, 3)),          # eight steps; image rows that do not fit one tile's LDS
    (1, 6, 7, 2, 18, 2, 3, (3, 3), (0, 4)),             # windows wholly in the padding
    (70, 24, 24, 3, 24, 3, 3, (1, 1), (1, 1)),          # enough tiles for four rows each, more than one per workgroup
    (260, 9, 20, 5, 96, 3, 1, (1, 1), (1, 0)),
]


@pytest.mark.parametrize("layout", ["krsc", "rsck"])
@pytest.mark.parametrize("case", CONVS)
def test_conv_few_channels(xp, oracle, case, layout):
    import torch
    n, h, w, ci, co, r, s, stride, pad = case
    x = inputs.to_bf16_bits(inputs.normal((n, h, w, ci), 0, 1))
    f = inputs.to_bf16_bits(inputs.normal((co, r, s, ci), 0, 2, (r * s * ci) ** -0.5))
    ref = oracle.conv2d_nhwc(x, f, N=n, H=h, W=w, Cin=ci, Cout=co, R=r, S=s, stride=stride, pad=pad)
    bad = x.copy()                                       # a pixel of NaNs belongs to the windows that hold it and to no other
    by, bx = h // 2, w // 2
    bad[n - 1, by, bx, :] = NAN_BITS
    hit = np.zeros(ref.shape[:3], bool)
    for p in range(ref.shape[1]):
        for q in range(ref.shape[2]):
            hit[n - 1, p, q] = 0 <= by - (p * stride[0] - pad[0]) < r and 0 <= bx - (q * stride[1] - pad[1]) < s
    flt = dev((f if layout == "krsc" else np.ascontiguousarray(f.transpose(1, 2, 3, 0))).reshape(-1))
    xp.xp_force_config(2, "bf16", _variant(xp, 2, "bf16", "few input channels"))
    for image in (x, bad):
        out = torch.full(ref.shape, 7.0, device="cuda")
        xp.xp_conv2d_nhwc(n, h, w, ci, co, r, s, *stride, *pad, dev(image.reshape(-1)), flt, layout, out, in_type="bf16", w_type="bf16")
        got = out.cpu().numpy()
        if image is bad:
            assert np.array_equal(np.isnan(got).all(-1), hit) and np.array_equal(np.isnan(got).any(-1), hit)
            check_float(got[~hit], ref[~hit], f"conv {case} {layout}, NaN elsewhere")
        else:
            check_float(got, ref, f"conv {case} {layout}")
    xp.xp_force_config(2, "bf16", -1)
