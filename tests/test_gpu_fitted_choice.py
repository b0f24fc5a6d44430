"""Calls where the fitted times displace the neighbouring table entry or the variants' own estimates, and calls that they leave
alone, asked with real buffers (the figures stand beside the rule).  The chosen kernel's result is checked against the general one's."""
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("batch,M,N,K,la,lb,text", [
    (0, 128, 512, 4352, "col", "row", "unaligned rows"),         # a long sum and few tiles: K shared out over a workgroup's waves
    (0, 384, 1152, 5696, "col", "row", "unaligned rows"),
    (0, 128, 512, 1024, "col", "row", "k-group-interleaved"),    # not so long
    (38, 640, 640, 128, "row", "col", "128x128x128B"),
    (104, 192, 192, 64, "row", "col", "stream"),
    (8, 752, 752, 64, "row", "col", "128B"),                     # too few rows of tiles to walk over columns
])
def test_fitted_choice(batch, M, N, K, la, lb, text):
    import torch
    from paper_2505_02146_amd import xp
    op, n = (1, batch) if batch else (0, 1)
    a, b = (torch.randint(-4, 5, (n * r * K,), device="cuda").bfloat16() for r in (M, N))
    lda, ldb = K if la == "row" else M, N if lb == "row" else K
    out = []
    for v in (-1, 0):                                            # integers: the general kernel's sums are exact too
        c = torch.full((n * M * N,), 7.0, device="cuda")
        xp.xp_force_config(op, "bf16", v)
        try:
            xp.xp_gemm_batched(n, M, N, K, 1.0, a, la, lda, M * K, b, lb, ldb, N * K, 0.0, c, "row", N, M * N) if batch else \
                xp.xp_gemm(M, N, K, 1.0, a, la, lda, b, lb, ldb, 0.0, c, "row", N)
            if v < 0:
                name = xp.xp_describe_config(op, "bf16", xp.xp_last_config(op, "bf16"))
        finally:
            xp.xp_force_config(op, "bf16", -1)
        out.append(c)
    assert torch.equal(*out)
    assert text in name, name
    assert ("stream" in text) == ("stream" in name), name
