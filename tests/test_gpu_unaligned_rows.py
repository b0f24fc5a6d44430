"""The GEMM-only tiles of the kernel for operands of any alignment (K groups, dealt-out loads, loads from dwords), forced at the
edges of tiles and K steps, against the oracle: int8 and integer-valued bf16 bit-exact (alpha, beta, batches), else the gates."""
import numpy as np
import pytest

from paper_2505_02146_amd import inputs
from tests.helpers import check_float, dev, store

pytestmark = pytest.mark.gpu

NAN_BITS = 0x7FC0
LAYOUTS = [("row", "col"), ("row", "row"), ("col", "row"), ("col", "col")]
# a step is 64 to 256 bf16 (128 to 512 int8) of K: K of 1 to 5 (rows around a dword), below one step, whole steps with one element
# more or less, several unchecked steps and a rest; extents around 32, 64, 96, 128 and 192, a single row and a single column
SHAPES = [(1, 17, 5), (33, 31, 1), (98, 33, 2), (97, 65, 3), (100, 97, 4), (129, 95, 5), (1, 40, 67), (50, 1, 259),
          (33, 31, 64), (97, 65, 257), (129, 95, 511), (193, 129, 1535), (64, 191, 2051), (96, 97, 2816)]


@pytest.fixture(scope="module")
def xp():
    from paper_2505_02146_amd import xp as m
    yield m
    for op in (0, 1):
        for t in ("bf16", "i8"):
            m.xp_force_config(op, t, -1)


def _forced(xp, op, kind):
    found = [v for v in range(xp.xp_num_configs(op, kind)) if "unaligned rows" in xp.xp_describe_config(op, kind, v)]
    assert len(found) == 6
    return found


def _taken(outer, K, along_k, ld, epc):
    """An operand of a chunk or more (epc elements); stored along its outer index, with a pitch of a chunk or more."""
    if along_k or ld == 1:
        return (outer - 1) * (ld if along_k else 1) + K >= epc
    return ld >= epc and (K - 1) * ld + outer >= epc


@pytest.mark.parametrize("kind", ["bf16", "i8"])
@pytest.mark.parametrize("la,lb", LAYOUTS)
def test_unaligned_rows(xp, oracle, kind, la, lb):
    import torch
    ran = 0
    for n, (M, N, K) in enumerate(SHAPES):
        for skew in (0, 1, 3):                           # elements in front of the operands: rows inside and on dwords
            make = (lambda s, t: inputs.int8_uniform(s, n, t)) if kind == "i8" else (lambda s, t: inputs.to_bf16_bits(inputs.normal(s, n, t)))
            fill = 99 if kind == "i8" else NAN_BITS      # what lies between the rows must not reach the result
            (a, lda), (b, ldb) = store(make((M, K), 1), la, (n + skew) % 4, fill), store(make((K, N), 2), lb, n % 3, fill)
            da, db = (dev(np.concatenate([x[:1].repeat(skew), x])) for x in (a, b))
            if kind == "i8":
                ref = oracle.gemm_i8(M, N, K, a, la, b, lb, lda=lda, ldb=ldb)
            else:
                ref = oracle.gemm_float(M, N, K, a, la, b, lb, lda=lda, ldb=ldb)
            for v in _forced(xp, 0, kind):
                xp.xp_force_config(0, kind, v)
                c = torch.full((M, N), 7, dtype=torch.int32 if kind == "i8" else torch.float32, device="cuda")
                what = f"{kind} {M}x{N}x{K} {la}/{lb} skew {skew} {xp.xp_describe_config(0, kind, v)}"
                epc = 16 if kind == "i8" else 8
                taken = _taken(M, K, la == "row", lda, epc) and _taken(N, K, lb == "col", ldb, epc)
                try:
                    xp.xp_gemm(M, N, K, 1.0, da[skew:], la, lda, db[skew:], lb, ldb, 0.0, c, "row", N, a_type=kind, b_type=kind)
                except xp.XpError as e:
                    assert e.status == 6 and not taken, what
                    continue
                finally:
                    xp.xp_force_config(0, kind, -1)
                assert taken, what
                ran += 1
                if kind == "i8":
                    assert np.array_equal(c.cpu().numpy(), ref), what
                else:
                    check_float(c.cpu().numpy(), ref, what)
    assert ran >= 3 * 6 * 11                             # of 14 shapes, three skews, six variants


@pytest.mark.parametrize("la,lb", LAYOUTS)
def test_unaligned_rows_batched(xp, oracle, la, lb):
    """Odd batch strides: the slices of a batch start on every byte of a dword; alpha and beta; nothing written between the slices."""
    import torch
    batch, M, N, K = 5, 67, 99, 645
    sA, sB, sC = M * K + 1, K * N + 3, M * N + 1
    A, B = (inputs.to_bf16_bits(inputs.small_integers((batch * s,), 1, t)) for s, t in ((sA, 1), (sB, 2)))
    lda, ldb = K if la == "row" else M, N if lb == "row" else K
    C0 = inputs.small_integers((batch * sC,), 1, 3)
    ref = oracle.gemm_float_batched(batch, M, N, K, A, la, B, lb, strideA=sA, strideB=sB)
    for v in _forced(xp, 1, "bf16"):
        xp.xp_force_config(1, "bf16", v)
        c = torch.from_numpy(C0.astype(np.float32)).cuda()
        try:
            xp.xp_gemm_batched(batch, M, N, K, 2.0, dev(A), la, lda, sA, dev(B), lb, ldb, sB, 3.0, c, "row", N, sC, a_type="bf16", b_type="bf16")
        finally:
            xp.xp_force_config(1, "bf16", -1)
        got = c.cpu().numpy().reshape(batch, sC)
        want = 2.0 * ref + 3.0 * C0.reshape(batch, sC)[:, :M * N].reshape(batch, M, N)
        assert np.array_equal(got[:, :M * N].reshape(batch, M, N), want), v
        assert np.array_equal(got[:, M * N:], C0.reshape(batch, sC)[:, M * N:]), "wrote between the slices"
