"""C with rows, bases and batch strides on every kind of boundary (4, 8, 16, 32 and 64 bytes): whole tiles, edges, both
store forms, against the oracle.  Integer-valued operands: every kernel has to give the oracle's value exactly."""
import numpy as np
import pytest

from paper_2505_02146_amd import inputs
from tests.helpers import dev

pytestmark = pytest.mark.gpu

VARIANTS = ["256x256x128B waves 2x2 ring 3(A)+2(B) direct-to-lds, reads as assembly, sub-steps paired",
            "256x256x128B waves 2x4 ring 3(A)+2(B) direct-to-lds, reads as assembly, mfma16",
            "256x256x128B waves 2x4 ring 2 direct-to-lds mfma16",
            "128x128x128B waves 2x2 ring 2(A)+2(B) direct-to-lds, reads as assembly, mfma16",
            "64x128-stream x128B single-k-step producer/consumer nt-stores"]


@pytest.mark.parametrize("kind", ["bf16", "i8"])
@pytest.mark.parametrize("pad,base", [(0, 0), (1, 0), (2, 3), (4, 0), (8, 4), (16, 8), (16, 0)])
@pytest.mark.parametrize("M,N", [(272, 264), (500, 511), (257, 385), (131, 254)])
def test_output_rows(oracle, kind, M, N, pad, base):
    """Whole tiles and edges that cut a wave's part, a block and four columns; `pad` elements between rows, `base` in front."""
    import torch
    from paper_2505_02146_amd import xp
    K, batch = 64, 2
    ldc = (N + 15) // 16 * 16 + pad                       # rows on 64 bytes where pad and base are multiples of 16
    if kind == "i8":
        A, B = (inputs.int8_uniform((batch, s, K), 5, t) for s, t in ((M, 1), (N, 2)))
    else:
        A, B = (inputs.to_bf16_bits(inputs.small_integers((batch, s, K), 5, t)) for s, t in ((M, 1), (N, 2)))
    ref = np.stack([oracle.gemm_i8(M, N, K, A[i], "row", B[i], "col") if kind == "i8" else oracle.gemm_float(M, N, K, A[i], "row", B[i], "col")
                    for i in range(batch)])
    a, b = dev(A), dev(B)
    stride = M * ldc + pad                                # (with pad 0: every slice on 64 bytes)
    names = [xp.xp_describe_config(1, kind, v) for v in range(xp.xp_num_configs(1, kind))]
    ran = set()
    for text in VARIANTS:
        for v in (i for i, n in enumerate(names) if text in n):
            for alpha, beta in ((1.0, 0.0),) if kind == "i8" else ((1.0, 0.0), (2.0, 0.0), (1.0, 3.0)):
                flat = torch.full((base + batch * stride,), 7, dtype=torch.int32 if kind == "i8" else torch.float32, device="cuda")
                xp.xp_force_config(1, kind, v)
                try:
                    xp.xp_gemm_batched(batch, M, N, K, alpha, a, "row", K, M * K, b, "col", K, N * K, beta, flat[base:], "row", ldc, stride,
                                       a_type=kind, b_type=kind)
                finally:
                    xp.xp_force_config(1, kind, -1)
                got = flat.cpu().numpy()
                assert np.all(got[:base] == 7)
                for i in range(batch):
                    c = got[base + i * stride:base + i * stride + M * ldc].reshape(M, ldc)
                    assert np.array_equal(c[:, :N], alpha * ref[i] + beta * 7), (names[v], alpha, beta)
                    assert np.all(c[:, N:] == 7), names[v]
                ran.add(text)
    assert ran == set(VARIANTS), "a variant of each kind"


# text, layouts, M, N: two tile heights (N of one tile: the two tiles of a compute unit in one workgroup; of three: in workgroups of
# their own), whose first part ends at a tile's edge and not the matrix's; operands along M and N
MORE = [("waves 2x4 ring 3(A)+2(B) direct-to-lds mfma16", "row", "col", 57644, 255), ("waves 2x4 ring 2(A)+2(B) direct-to-lds, reads as assembly", "row", "col", 57644, 253),
        ("waves 2x2 ring 3(A)+2(B) direct-to-lds, reads as assembly, sub-steps paired", "row", "col", 57644, 254),
        ("waves 2x4 ring 2(A)+2(B) direct-to-lds, reads as assembly", "row", "col", 38330, 513),
        ("waves 2x2 ring 3(A)+2(B) direct-to-lds, reads as assembly, sub-steps paired", "row", "col", 38330, 515)]
MORE = [("224x256x128B then 192x256 in the last round, " + text, *rest) for text, *rest in MORE] + [
    (f"{tile} direct-to-lds, {along} by transposing reads", la, lb, 504, 488)
    for along, la, lb in (("B along N", "row", "row"), ("A along M", "col", "col"), ("A along M and B along N", "col", "row"))
    for tile in ("256x256x128B waves 2x2 ring 3(A)+2(B)", "256x256x128B waves 2x4 ring 2(A)+2(B)", "256x128x128B waves 4x2 ring 3(A)+3(B)",
                 "128x128x128B waves 2x2 ring 2(A)+2(B)")]


@pytest.mark.parametrize("text,la,lb,M,N", MORE)
@pytest.mark.parametrize("pad,base", [(0, 0), (1, 0), (5, 3), (None, 0)])
def test_output_rows_of_two_heights_and_transposing_reads(text, la, lb, M, N, pad, base):
    """The same ends of C in these kernels (pad None: rows on 64 bytes), against the general kernel; integers, so exact."""
    import torch
    from paper_2505_02146_amd import xp
    K = 72                                                # a K step and a rest
    ldc = (N + 15) // 16 * 16 if pad is None else N + pad
    a, b = (torch.randint(-3, 4, (r * K,), device="cuda").bfloat16() for r in (M, N))
    names = [xp.xp_describe_config(0, "bf16", v) for v in range(xp.xp_num_configs(0, "bf16"))]
    found = [v for v, n in enumerate(names) if text in n]
    assert len(found) == 1, (text, found)

    def run(v, alpha, beta):
        flat = torch.full((base + M * ldc + 64,), 7.0, device="cuda")
        xp.xp_force_config(0, "bf16", v)
        try:
            xp.xp_gemm(M, N, K, alpha, a, la, K if la == "row" else M, b, lb, N if lb == "row" else K, beta, flat[base:], "row", ldc)
        finally:
            xp.xp_force_config(0, "bf16", -1)
        return flat

    for alpha, beta in ((1.0, 0.0), (2.0, 0.0), (1.0, 3.0)):
        assert torch.equal(run(found[0], alpha, beta), run(0, alpha, beta)), (names[found[0]], alpha, beta)
