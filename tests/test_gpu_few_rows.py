"""The kernel for few rows against a large matrix, forced at the edges of its blocks and steps, against the oracle (int8
bit-exact, bf16 the gates)."""
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


def _variant(xp, op, kind, text):
    found = [v for v in range(xp.xp_num_configs(op, kind)) if text in xp.xp_describe_config(op, kind, v)]
    assert len(found) == 1
    return found[0]


# rows of X: one block, its edges, two and four blocks; W around its 16 / 32-row blocks; K below one block of 128 bytes, whole
# blocks (fewer and more than the eight waves, the prefetch's remainder) and ragged ends; 8200 rows take 32 a workgroup
FEW = [(1, 33, 70), (3, 16, 64), (16, 100, 1024), (17, 65, 1111), (33, 40, 5000), (64, 31, 4096), (16, 8200, 520), (5, 8210, 131), (40, 8193, 200)]


@pytest.mark.parametrize("kind", ["bf16", "i8"])
@pytest.mark.parametrize("few_columns", [False, True])
def test_few_rows(xp, oracle, kind, few_columns):
    """few_columns: the few are columns of a row-major C, i.e. W is the first operand."""
    import torch
    v = _variant(xp, 0, kind, "few rows")
    for n, (few, many, K) in enumerate(FEW):
        M, N = (many, few) if few_columns else (few, many)
        make = (lambda s, t: inputs.int8_uniform(s, n, t)) if kind == "i8" else (lambda s, t: inputs.to_bf16_bits(inputs.normal(s, n, t)))
        fill = 99 if kind == "i8" else NAN_BITS
        (a, lda), (b, ldb) = store(make((M, K), 1), "row", n % 3, fill), store(make((K, N), 2), "col", n % 2, fill)
        if kind == "i8":
            ref = oracle.gemm_i8(M, N, K, a, "row", b, "col", lda=lda, ldb=ldb)
        else:
            ref = oracle.gemm_float(M, N, K, a, "row", b, "col", lda=lda, ldb=ldb)
        xp.xp_force_config(0, kind, v)
        ldc = N + n % 2
        c = torch.full((M, ldc), 7, dtype=torch.int32 if kind == "i8" else torch.float32, device="cuda")
        xp.xp_gemm(M, N, K, 1.0, dev(a), "row", lda, dev(b), "col", ldb, 0.0, c, "row", ldc, a_type=kind, b_type=kind)
        xp.xp_force_config(0, kind, -1)
        got = c.cpu().numpy()
        what = f"{kind} {M}x{N}x{K}"
        assert np.all(got[:, N:] == 7), what + " wrote into the ld padding"
        if kind == "i8":
            assert np.array_equal(got[:, :N], ref), what
        else:
            check_float(got[:, :N], ref, what)


def test_few_rows_alpha_beta_batched(xp, oracle):
    import torch
    v = _variant(xp, 1, "bf16", "few rows")
    batch, M, N, K = 3, 20, 50, 300
    A, B = (inputs.to_bf16_bits(inputs.small_integers((batch * s,), 1, t)) for s, t in ((M * K, 1), (N * K, 2)))
    C0 = inputs.small_integers((batch, M, N), 1, 3).astype(np.float32)
    ref = oracle.gemm_float_batched(batch, M, N, K, A, "row", B, "col")
    c = torch.from_numpy(C0).cuda()
    xp.xp_force_config(1, "bf16", v)
    xp.xp_gemm_batched(batch, M, N, K, 2.0, dev(A), "row", K, M * K, dev(B), "col", K, N * K, 3.0, c, "row", N, M * N, a_type="bf16", b_type="bf16")
    xp.xp_force_config(1, "bf16", -1)
    assert np.array_equal(c.cpu().numpy(), 2.0 * ref + 3.0 * C0)



# 17 to 64 rows of X against as many rows of W as make workgroups of 24, 32 and 40 of them, the last one ragged
@pytest.mark.parametrize("kind", ["bf16", "i8"])
@pytest.mark.parametrize("few,many,K", [(24, 6001, 300), (20, 10001, 1100), (33, 6008, 520), (48, 10003, 264), (41, 8180, 1111), (64, 6010, 500)])
def test_few_rows_splits(xp, oracle, kind, few, many, K):
    import torch
    make = (lambda s, t: inputs.int8_uniform(s, 1, t)) if kind == "i8" else (lambda s, t: inputs.to_bf16_bits(inputs.normal(s, 1, t)))
    (a, lda), (b, ldb) = store(make((few, K), 1), "row"), store(make((K, many), 2), "col")
    ref = oracle.gemm_i8(few, many, K, a, "row", b, "col") if kind == "i8" else oracle.gemm_float(few, many, K, a, "row", b, "col")
    c = torch.full((few, many), 7, dtype=torch.int32 if kind == "i8" else torch.float32, device="cuda")
    xp.xp_force_config(0, kind, _variant(xp, 0, kind, "few rows"))
    xp.xp_gemm(few, many, K, 1.0, dev(a), "row", lda, dev(b), "col", ldb, 0.0, c, "row", many, a_type=kind, b_type=kind)
    xp.xp_force_config(0, kind, -1)
    if kind == "i8":
        assert np.array_equal(c.cpu().numpy(), ref)
    else:
        check_float(c.cpu().numpy(), ref, f"{few}x{many}x{K}")


@pytest.mark.parametrize("kind", ["bf16", "i8"])
@pytest.mark.parametrize("few", [3, 17])
def test_few_rows_of_a_streamed_matrix(xp, oracle, kind, few):
    """W of 64 MB and more takes loads of its own; odd K, a ragged last workgroup."""
    many, K = 8201, 8209 if kind == "i8" else 4105
    assert many * K * (1 if kind == "i8" else 2) >= 64 << 20
    import torch
    make = (lambda s, t: inputs.int8_uniform(s, 1, t)) if kind == "i8" else (lambda s, t: inputs.to_bf16_bits(inputs.normal(s, 1, t)))
    A, B = make((few, K), 1), make((many, K), 2)
    ref = oracle.gemm_i8(few, many, K, A.reshape(-1), "row", B.reshape(-1), "col") if kind == "i8" else oracle.gemm_float(few, many, K, A.reshape(-1), "row", B.reshape(-1), "col")
    c = torch.full((few, many), 7, dtype=torch.int32 if kind == "i8" else torch.float32, device="cuda")
    xp.xp_force_config(0, kind, _variant(xp, 0, kind, "few rows"))
    xp.xp_gemm(few, many, K, 1.0, dev(A.reshape(-1)), "row", K, dev(B.reshape(-1)), "col", K, 0.0, c, "row", many, a_type=kind, b_type=kind)
    xp.xp_force_config(0, kind, -1)
    if kind == "i8":
        assert np.array_equal(c.cpu().numpy(), ref)
    else:
        check_float(c.cpu().numpy(), ref, f"{few}x{many}x{K}")
