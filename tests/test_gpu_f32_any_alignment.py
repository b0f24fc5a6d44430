"""The small fp32 kernel's 16-byte loads at any alignment, forced at the edges of groups, chunks and tiles, against the oracle."""
import numpy as np
import pytest

from paper_2505_02146_amd import inputs
from tests.helpers import check_float, dev, store

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def xp():
    from paper_2505_02146_amd import xp as m
    yield m
    for op in (0, 1):
        m.xp_force_config(op, "f32", -1)


def _variant(xp, op):
    found = [v for v in range(xp.xp_num_configs(op, "f32")) if "four waves split k" in xp.xp_describe_config(op, "f32", v)]
    assert len(found) == 1
    return found[0]


# one group that is the operand, groups that stick out by 1 to 3, K around a chunk of 256 and several, tiles of 32 and their edges
SHAPES = [(2, 3, 2), (4, 1, 4), (33, 31, 257), (32, 64, 255), (17, 65, 513), (5, 39, 770), (66, 3, 1), (3, 130, 1023)]


@pytest.mark.parametrize("a_l", ["row", "col"])
@pytest.mark.parametrize("b_l", ["row", "col"])
def test_f32_any_alignment(xp, oracle, a_l, b_l):
    import torch
    for n, (M, N, K) in enumerate(SHAPES):
        A, B = inputs.normal((M, K), n, 1), inputs.normal((K, N), n, 2)
        (a, lda), (b, ldb) = store(A, a_l, n % 3, np.nan), store(B, b_l, n % 2, np.nan)
        ref = oracle.gemm_float(M, N, K, a, a_l, b, b_l, lda=lda, ldb=ldb)
        ldc = N + n % 2
        c = torch.full((M, ldc), 7.0, device="cuda")
        xp.xp_force_config(0, "f32", _variant(xp, 0))
        # operands that start one element past a 16-byte boundary, with NaNs around them
        ax, bx = (dev(np.concatenate([np.full(1, np.nan, np.float32), v, np.full(1, np.nan, np.float32)])) for v in (a, b))
        xp.xp_gemm(M, N, K, 1.0, ax[1:], a_l, lda, bx[1:], b_l, ldb, 0.0, c, "row", ldc)
        xp.xp_force_config(0, "f32", -1)
        got = c.cpu().numpy()
        assert np.all(got[:, N:] == 7), "wrote into the ld padding"
        check_float(got[:, :N], ref, f"f32 {M}x{N}x{K} {a_l} {b_l}")


def test_f32_any_alignment_alpha_beta_batched(xp, oracle):
    import torch
    batch, M, N, K = 3, 19, 35, 301
    A, B = (inputs.small_integers((batch * s,), 1, t).astype(np.float32) for s, t in ((M * K, 1), (N * K, 2)))
    C0 = inputs.small_integers((batch, M, N), 1, 3).astype(np.float32)
    ref = oracle.gemm_float_batched(batch, M, N, K, A, "row", B, "col")
    c = torch.from_numpy(C0).cuda()
    xp.xp_force_config(1, "f32", _variant(xp, 1))
    xp.xp_gemm_batched(batch, M, N, K, 2.0, dev(A), "row", K, M * K, dev(B), "col", K, N * K, 3.0, c, "row", N, M * N)
    xp.xp_force_config(1, "f32", -1)
    assert np.array_equal(c.cpu().numpy(), 2.0 * ref + 3.0 * C0)
