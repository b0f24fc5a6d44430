"""The MFMA kernel for operands of any alignment: every tile variant forced on extents, pitches and offsets that are no
multiple of a 16-byte chunk, against the oracle.  Bounds: int8 and integer-valued bf16 bit-exact, else the gates."""
import numpy as np
import pytest

from paper_2505_02146_amd import inputs
from tests.helpers import check_float, dev, store

pytestmark = pytest.mark.gpu

NAN_BITS = 0x7FC0


@pytest.fixture(scope="module")
def xp():
    from paper_2505_02146_amd import xp as m
    yield m
    for op in (0, 1, 2):
        for t in ("bf16", "i8"):
            m.xp_force_config(op, t, -1)


def _forced(xp, op, kind):
    names = [xp.xp_describe_config(op, kind, v) for v in range(xp.xp_num_configs(op, kind))]
    found = [v for v, n in enumerate(names) if "any alignment" in n]
    assert len(found) == 3
    return found


# extents around a chunk, an MFMA block, a tile and a K step (64 bf16 / 128 int8), none of them aligned; the last row has
# several tiles of every size and several unchecked steps
SHAPES = [(1, 9, 1), (17, 16, 7), (63, 65, 65), (65, 129, 127), (130, 131, 129), (127, 257, 191), (261, 200, 395)]


@pytest.mark.parametrize("kind", ["bf16", "i8"])
@pytest.mark.parametrize("la,lb", [("row", "col"), ("row", "row"), ("col", "row"), ("col", "col")])
def test_gemm_any_alignment(xp, oracle, kind, la, lb):
    import torch
    for n, (M, N, K) in enumerate(SHAPES):
        skew = n % 3                                     # the operands start 0, 1, 2 elements past an aligned address
        make = (lambda s, t: inputs.int8_uniform(s, n, t)) if kind == "i8" else (lambda s, t: inputs.to_bf16_bits(inputs.normal(s, n, t)))
        fill = 99 if kind == "i8" else NAN_BITS          # what lies between the rows must not reach the result
        (a, lda), (b, ldb) = store(make((M, K), 1), la, n % 4, fill), store(make((K, N), 2), lb, n % 3, fill)
        da, db = (dev(np.concatenate([x[:1].repeat(skew), x])) for x in (a, b))
        if kind == "i8":
            ref = oracle.gemm_i8(M, N, K, a, la, b, lb, lda=lda, ldb=ldb)
        else:
            ref = oracle.gemm_float(M, N, K, a, la, b, lb, lda=lda, ldb=ldb)
        for v in _forced(xp, 0, kind):
            xp.xp_force_config(0, kind, v)
            c = torch.full((M, N), 7, dtype=torch.int32 if kind == "i8" else torch.float32, device="cuda")
            try:
                xp.xp_gemm(M, N, K, 1.0, da[skew:], la, lda, db[skew:], lb, ldb, 0.0, c, "row", N, a_type=kind, b_type=kind)
            except xp.XpError as e:                      # an operand or a pitch along M or N below one chunk is declined
                small = min(M, N) * K < 16 or (la == "col" and lda < 16) or (lb == "row" and ldb < 16)
                assert e.status == 6 and small, (M, N, K, la, lb)
                continue
            what = f"{kind} {M}x{N}x{K} {la}/{lb} skew {skew} variant {v}"
            if kind == "i8":
                assert np.array_equal(c.cpu().numpy(), ref), what
            else:
                check_float(c.cpu().numpy(), ref, what)
        xp.xp_force_config(0, kind, -1)


def test_batched_odd_strides_alpha_beta(xp, oracle):
    import torch
    batch, M, N, K = 3, 67, 45, 99
    sA, sB, sC = M * K + 3, K * N + 5, M * N + 1
    A, B = (inputs.to_bf16_bits(inputs.small_integers((batch * s,), 1, t)) for s, t in ((sA, 1), (sB, 2)))
    C0 = inputs.small_integers((batch * sC,), 1, 3)
    ref = oracle.gemm_float_batched(batch, M, N, K, A, "row", B, "row", strideA=sA, strideB=sB)
    for v in _forced(xp, 1, "bf16"):
        xp.xp_force_config(1, "bf16", v)
        c = torch.from_numpy(C0.astype(np.float32)).cuda()
        xp.xp_gemm_batched(batch, M, N, K, 2.0, dev(A), "row", K, sA, dev(B), "row", N, sB, 3.0, c, "row", N, sC, a_type="bf16", b_type="bf16")
        got = c.cpu().numpy().reshape(batch, sC)
        want = 2.0 * ref + 3.0 * C0.reshape(batch, sC)[:, :M * N].reshape(batch, M, N)
        assert np.array_equal(got[:, :M * N].reshape(batch, M, N), want), v
        assert np.array_equal(got[:, M * N:], C0.reshape(batch, sC)[:, M * N:]), "wrote between the slices"
    xp.xp_force_config(1, "bf16", -1)


CONVS = [
    # N, H, W, Cin, Cout, R, S, stride, pad
    (2, 19, 23, 3, 64, 7, 7, (2, 2), (3, 3)),           # a first layer: runs of 21 elements
    (1, 5, 6, 1, 9, 3, 3, (1, 1), (1, 1)),              # runs of 3: one chunk each, the whole image smaller than a tile
    (2, 9, 8, 5, 70, 3, 5, (1, 2), (2, 4)),             # windows that stick out on both sides
    (1, 11, 7, 40, 33, 1, 1, (1, 1), (0, 0)),           # one run
    (2, 13, 12, 34, 129, 3, 3, (1, 1), (1, 1)),         # runs of 102
    (1, 4, 300, 2, 17, 2, 1, (1, 1), (0, 3)),           # one column of taps, padding beyond the filter's width
]


@pytest.mark.parametrize("layout", ["krsc", "rsck"])
@pytest.mark.parametrize("case", CONVS)
def test_conv_any_channel_count(xp, oracle, case, layout):
    import torch
    n, h, w, ci, co, r, s, stride, pad = case
    x = inputs.to_bf16_bits(inputs.normal((n, h, w, ci), 0, 1))
    f = inputs.to_bf16_bits(inputs.normal((co, r, s, ci), 0, 2, (r * s * ci) ** -0.5))
    ref = oracle.conv2d_nhwc(x, f, N=n, H=h, W=w, Cin=ci, Cout=co, R=r, S=s, stride=stride, pad=pad)
    # one pixel of NaNs: they belong to the windows that hold the pixel and to no other (a masked element counts for nothing)
    bad = x.copy()
    bad[n - 1, h // 2, w // 2, :] = NAN_BITS
    hit = np.zeros(ref.shape[:3], bool)
    for p in range(ref.shape[1]):
        for q in range(ref.shape[2]):
            y0, x0 = p * stride[0] - pad[0], q * stride[1] - pad[1]
            hit[n - 1, p, q] = y0 <= h // 2 < y0 + r and x0 <= w // 2 < x0 + s
    flt = dev((f if layout == "krsc" else np.ascontiguousarray(f.transpose(1, 2, 3, 0))).reshape(-1))
    for v in _forced(xp, 2, "bf16"):
        xp.xp_force_config(2, "bf16", v)
        for image in (x, bad):
            out = torch.full(ref.shape, 7.0, device="cuda")
            xp.xp_conv2d_nhwc(n, h, w, ci, co, r, s, *stride, *pad, dev(image.reshape(-1)), flt, layout, out, in_type="bf16", w_type="bf16")
            got = out.cpu().numpy()
            if image is bad:
                assert np.array_equal(np.isnan(got).all(-1), hit) and np.array_equal(np.isnan(got).any(-1), hit), (case, layout, v)
                check_float(got[~hit], ref[~hit], f"conv {case} {layout} variant {v}, NaN elsewhere")
            else:
                check_float(got, ref, f"conv {case} {layout} variant {v}")
    xp.xp_force_config(2, "bf16", -1)


def test_selection_takes_the_matrix_cores(xp, oracle):
    """Calls that no aligned kernel takes no longer end on the general kernel."""
    import torch
    z = torch.zeros(1 << 16, dtype=torch.int16, device="cuda")
    c = torch.zeros(1 << 16, device="cuda")
    xp.xp_gemm(100, 101, 99, 1.0, z, "row", 99, z, "row", 101, 0.0, c, "row", 101, a_type="bf16", b_type="bf16")
    assert "any alignment" in xp.xp_describe_config(0, "bf16", xp.xp_last_config(0, "bf16"))
    xp.xp_conv2d_nhwc(1, 16, 16, 34, 32, 3, 3, 1, 1, 1, 1, z, z, "krsc", c, in_type="bf16", w_type="bf16")
    assert "any alignment" in xp.xp_describe_config(2, "bf16", xp.xp_last_config(2, "bf16"))
