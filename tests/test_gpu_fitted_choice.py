"""Calls where the fitted times displace the neighbouring table entry or the variants' own estimates, and calls that they leave
alone, asked with real buffers (the figures stand beside the rule).  The chosen kernel's result is checked against the general one's."""
import pytest

pytestmark = pytest.mark.gpu


def _run(kind, batch, M, N, K, la, lb):
    """The name of the variant that was chosen; its result has to be the general kernel's."""
    import torch
    from paper_2505_02146_amd import xp
    op, n = (1, batch) if batch else (0, 1)
    a, b = (torch.randint(-4, 5, (n * r * K,), device="cuda").to(torch.bfloat16 if kind == "bf16" else torch.int8) for r in (M, N))
    lda, ldb = K if la == "row" else M, N if lb == "row" else K
    out = []
    for v in (-1, 0):                                            # integers: the general kernel's sums are exact too
        c = torch.full((n * M * N,), 7, device="cuda", dtype=torch.float32 if kind == "bf16" else torch.int32)
        xp.xp_force_config(op, kind, v)
        try:
            xp.xp_gemm_batched(n, M, N, K, 1.0, a, la, lda, M * K, b, lb, ldb, N * K, 0.0, c, "row", N, M * N) if batch else \
                xp.xp_gemm(M, N, K, 1.0, a, la, lda, b, lb, ldb, 0.0, c, "row", N)
            if v < 0:
                name = xp.xp_describe_config(op, kind, xp.xp_last_config(op, kind))
        finally:
            xp.xp_force_config(op, kind, -1)
        out.append(c)
    assert torch.equal(*out)
    return name


@pytest.mark.parametrize("batch,M,N,K,la,lb,text", [
    (0, 128, 512, 4352, "col", "row", "unaligned rows"),         # a long sum and few tiles: K shared out over a workgroup's waves
    (0, 384, 1152, 5696, "col", "row", "unaligned rows"),
    (0, 128, 512, 1024, "col", "row", "k-group-interleaved"),    # not so long
    (38, 640, 640, 128, "row", "col", "128x128x128B"),
    (104, 192, 192, 64, "row", "col", "stream"),
    (8, 752, 752, 64, "row", "col", "128B"),                     # too few rows of tiles to walk over columns
])
def test_fitted_choice(batch, M, N, K, la, lb, text):
    name = _run("bf16", batch, M, N, K, la, lb)
    assert text in name, name
    assert ("stream" in text) == ("stream" in name), name


@pytest.mark.parametrize("kind,batch,M,N,K,la,lb,text", [
    ("bf16", 0, 4096, 4096, 4032, "col", "col", "256x256"), ("bf16", 0, 4096, 4096, 1088, "col", "col", "256x256"),
    ("bf16", 0, 2048, 8192, 1088, "col", "col", "256x256"), ("bf16", 0, 4096, 4096, 4032, "col", "row", "256x256"),
    ("bf16", 0, 3072, 3072, 3008, "col", "row", "256x256"), ("bf16", 0, 1632, 6624, 592, "col", "col", "256x256"),
    ("bf16", 0, 1536, 8192, 4160, "row", "col", "224x256"),
    ("i8", 96, 512, 512, 64, "row", "col", "64x64-stream"), ("i8", 96, 512, 512, 128, "row", "col", "64x64-stream"),
    ("i8", 32, 1024, 1024, 128, "row", "col", "64x64-stream"),
])
def test_a_choice_without_a_fitted_time_stands(kind, batch, M, N, K, la, lb, text):
    """Neighbours of swept shapes whose winners were timed faster than every variant with a fitted time."""
    name = _run(kind, batch, M, N, K, la, lb)
    assert text in name, name


@pytest.mark.parametrize("kind,batch,M,N,K,la,lb,text", [
    # rows that the timings refuted are no candidates: the choice stands ...
    ("bf16", 0, 2304, 5800, 504, "col", "row", "256x256x128B"), ("bf16", 0, 1768, 640, 64, "row", "row", "128x64x128B"),
    ("i8", 0, 6784, 272, 224, "col", "col", "64x64x128B"), ("i8", 7, 528, 528, 64, "row", "row", "64x64x128B"),
    # ... and others displace it
    ("i8", 0, 256, 256, 8192, "col", "row", "unaligned rows"), ("i8", 0, 208, 416, 6144, "row", "row", "unaligned rows"),
])
def test_candidates(kind, batch, M, N, K, la, lb, text):
    name = _run(kind, batch, M, N, K, la, lb)
    assert text in name, name


@pytest.mark.parametrize("kind,batch,M,N,K,la,lb,text", [
    # tiles for rows on any element, A along M: what that adds to a step
    ("i8", 0, 1280, 256, 6584, "col", "col", "64x32 waves"), ("i8", 0, 140, 148, 5132, "col", "col", "64x32 waves"),
    ("i8", 0, 7731, 1896, 3102, "col", "col", "128x128x128B waves 2x2 any"), ("i8", 0, 1132, 4680, 6776, "col", "row", "192x128"),
    ("i8", 61, 134, 134, 128, "col", "row", "64x64x128B waves 2x2 any"), ("bf16", 26, 410, 129, 414, "col", "col", "64x64x128B waves 2x2 any"),
    ("bf16", 159, 769, 128, 769, "col", "col", "128x128x128B waves 2x2 any"),
    ("bf16", 0, 2049, 1021, 1535, "row", "row", "96x96"),
])
def test_choice_of_tiles_for_any_alignment(kind, batch, M, N, K, la, lb, text):
    name = _run(kind, batch, M, N, K, la, lb)
    assert text in name, name


@pytest.mark.parametrize("n,h,cin,cout,r,stride,pad,text", [
    (53, 14, 32, 272, 1, 1, 0, "128x128x64B"), (3, 112, 32, 328, 1, 2, 0, "128x128x64B"), (27, 112, 320, 192, 1, 2, 0, "224x256x128B"),
    (4, 112, 320, 53, 5, 1, 2, "256x128x128B waves 4x2"),
])
def test_candidates_of_convolutions(n, h, cin, cout, r, stride, pad, text):
    import torch
    from paper_2505_02146_amd import xp
    x, f = (torch.randint(-2, 3, (e,), device="cuda").bfloat16() for e in (n * h * h * cin, cout * r * r * cin))
    P, out = (h + 2 * pad - r) // stride + 1, []
    for v in (-1, 0):
        c = torch.full((n * P * P * cout,), 7.0, device="cuda")
        xp.xp_force_config(2, "bf16", v)
        try:
            xp.xp_conv2d_nhwc(n, h, h, cin, cout, r, r, stride, stride, pad, pad, x, f, "krsc", c)
            if v < 0:
                name = xp.xp_describe_config(2, "bf16", xp.xp_last_config(2, "bf16"))
        finally:
            xp.xp_force_config(2, "bf16", -1)
        out.append(c)
    assert torch.equal(*out)
    assert text in name, name
