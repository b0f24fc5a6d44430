"""Which kernel the library picks where several can run the call: lines that were measured on both sides (the figures stand
beside the rules), asked with real buffers."""
import pytest

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def xp():
    from paper_2505_02146_amd import xp as m
    for op in (0, 1, 2):
        for t in ("f32", "bf16", "i8"):
            m.xp_force_config(op, t, -1)
    return m


_TORCH = {"f32": "float32", "bf16": "bfloat16", "i8": "int8"}


def _gemm(xp, kind, batch, M, N, K, la="row", lb="col", skew=0):
    """The name of the kernel that a product with operands `skew` elements past an aligned address ran on."""
    import torch
    n = max(batch, 1)
    a, b = (torch.zeros(n * r * K + skew, dtype=getattr(torch, _TORCH[kind]), device="cuda")[skew:] for r in (M, N))
    c = torch.full((n * M * N,), 7, dtype=torch.int32 if kind == "i8" else torch.float32, device="cuda")
    lda, ldb = (K if la == "row" else M), (N if lb == "row" else K)
    if batch == 0:
        xp.xp_gemm(M, N, K, 1.0, a, la, lda, b, lb, ldb, 0.0, c, "row", N)
    else:
        xp.xp_gemm_batched(batch, M, N, K, 1.0, a, la, lda, M * K, b, lb, ldb, N * K, 0.0, c, "row", N, M * N)
    assert not c.any(), "zeros times zeros"
    op = 0 if batch == 0 else 1
    return xp.xp_describe_config(op, kind, xp.xp_last_config(op, kind))


@pytest.mark.parametrize("kind", ["bf16", "i8"])
@pytest.mark.parametrize("call,few", [
    ((0, 16, 8192, 2048), True), ((0, 64, 4096, 4096), True), ((0, 40, 2560, 8192), True), ((0, 20, 10240, 4096), True), ((2, 4, 1024, 1024), True),
    # many problems: a workgroup per 64-row tile of the other kernels is more than the chip holds at once
    ((96, 64, 687, 32), False), ((192, 64, 1024, 64), False), ((96, 49, 6144, 48), False), ((32, 33, 4096, 512), False),
    ((128, 17, 256, 2048), False), ((128, 1024, 7, 64), False), ((128, 64, 64, 4096), False), ((0, 64, 16384, 2048), False),
    # rows off a 16-byte boundary: more than 48 rows against more than 32 tiles stay with the any-alignment kernel
    ((0, 64, 6976, 6913), False), ((0, 49, 2112, 6913), False), ((0, 48, 6976, 6913), True), ((0, 64, 1728, 6913), True), ((0, 64, 6976, 6912), True),
])
def test_few_rows(xp, kind, call, few):
    assert ("few rows" in _gemm(xp, kind, *call)) == few


@pytest.mark.parametrize("call,small", [
    ((0, 61, 1021, 130), True), ((0, 257, 255, 20001), True), ((0, 1001, 1003, 1005), True), ((0, 500, 1001, 377), True),
    ((0, 132, 4926, 377), False), ((0, 2001, 2003, 701), False), ((48, 112, 569, 251), False), ((0, 4001, 4003, 129), False),
])
@pytest.mark.parametrize("la,lb", [("row", "col"), ("row", "row"), ("col", "col")])
def test_fp32_kernel_for_small_products(xp, call, small, la, lb):
    """Operands of any alignment: 32x32 tiles up to four per compute unit, the tiled kernels beyond."""
    assert ("four waves split k" in _gemm(xp, "f32", *call, la=la, lb=lb, skew=1)) == small


def _conv(xp, call, layout="krsc"):
    """The name of the kernel that a convolution ran on (N, H, W, Cin, Cout, R, S, stride, pad)."""
    import torch
    n, h, w, ci, co, r, s, st, p = call
    x, f = (torch.zeros(e, dtype=torch.bfloat16, device="cuda") for e in (n * h * w * ci, co * r * s * ci))
    ph, pw = (p, p) if h > 1 else (0, p)
    P, Q = (h + 2 * ph - r) // st + 1, (w + 2 * pw - s) // st + 1
    out = torch.full((n * P * Q * co,), 7.0, device="cuda")
    xp.xp_conv2d_nhwc(n, h, w, ci, co, r, s, st, st, ph, pw, x, f, layout, out)
    assert not out.any()
    return xp.xp_describe_config(2, "bf16", xp.xp_last_config(2, "bf16"))


@pytest.mark.parametrize("call,any_alignment", [
    # N, H, W, Cin, Cout, R, S, stride, pad
    ((6, 7, 7, 256, 32, 11, 11, 1, 5), False), ((2, 1, 1434, 64, 32, 1, 40, 2, 0), False), ((1, 28, 28, 64, 176, 7, 7, 2, 3), False),
    ((1, 28, 28, 32, 176, 7, 7, 2, 3), True),            # 64-byte pixels and more than 32 taps
    ((1, 28, 28, 72, 176, 7, 7, 2, 3), True), ((1, 28, 28, 64, 176, 3, 3, 1, 1), False),
])
def test_convolutions_of_many_taps(xp, call, any_alignment):
    assert ("any alignment" in _conv(xp, call)) == any_alignment


@pytest.mark.parametrize("call,layout,few", [
    ((8, 224, 224, 3, 64, 7, 7, 2, 3), "krsc", True), ((2, 224, 224, 3, 64, 3, 3, 1, 1), "krsc", True),
    ((8, 224, 224, 3, 64, 7, 7, 2, 3), "rsck", False), ((16, 120, 120, 3, 32, 3, 3, 1, 1), "rsck", True),
    ((2, 37, 30, 3, 64, 7, 7, 2, 3), "krsc", False), ((2, 60, 60, 3, 4, 3, 3, 1, 1), "rsck", True),
    ((2, 1, 7427, 1, 128, 1, 15, 1, 0), "krsc", False), ((9, 1, 20066, 1, 4, 1, 40, 1, 0), "krsc", False),
    ((4, 1, 4261, 2, 4, 1, 3, 1, 0), "rsck", False), ((19, 1, 4930, 7, 4, 1, 15, 2, 0), "rsck", True),
    ((16, 60, 60, 6, 448, 3, 3, 1, 1), "krsc", True), ((16, 60, 60, 6, 448, 3, 3, 1, 1), "rsck", False),
    ((34, 1, 20000, 6, 8, 1, 5, 2, 0), "krsc", True), ((14, 1, 33664, 1, 16, 1, 1, 1, 0), "krsc", False),
])
def test_convolutions_of_few_channels(xp, call, layout, few):
    assert ("few input channels" in _conv(xp, call, layout)) == few


def _fresh(call):
    """`call` in a thread of its own, which remembers no selection."""
    import threading
    box = []
    t = threading.Thread(target=lambda: box.append(call()))
    t.start()
    t.join()
    return box[0]


@pytest.mark.parametrize("kind,call,la,lb", [
    ("bf16", (0, 512, 384, 512), "row", "col"), ("bf16", (0, 512, 384, 512), "row", "row"), ("i8", (0, 512, 384, 512), "row", "col"),
    ("bf16", (0, 5120, 1, 1024), "row", "col"), ("bf16", (0, 32, 10240, 4096), "row", "col"), ("f32", (0, 768, 512, 512), "row", "col"),
    ("bf16", (3, 256, 128, 256), "row", "col"),
])
def test_a_remembered_choice_is_for_its_alignment_only(xp, kind, call, la, lb):
    """Misaligned operands, then aligned ones of the same shape, and the other way round: what a first call would run."""
    aligned, off = (_fresh(lambda s=s: _gemm(xp, kind, *call, la=la, lb=lb, skew=s)) for s in (0, 1))
    assert aligned != off, "the case is meant to be one where alignment decides"
    for skew in (1, 0, 1, 1, 0, 0):
        assert _gemm(xp, kind, *call, la=la, lb=lb, skew=skew) == (off if skew else aligned), skew


def test_a_tuned_choice_is_for_its_alignment_only(xp, tmp_path):
    import torch
    M, N, K = 512, 384, 512
    xp.xp_tune_clear()
    aligned = _fresh(lambda: _gemm(xp, "bf16", 0, M, N, K))
    ws = torch.empty(xp.xp_tune_workspace_bytes(M * N), dtype=torch.uint8, device="cuda")
    a, b = (torch.randn(r * K + 1, device="cuda").bfloat16()[1:] for r in (M, N))
    c = torch.zeros(M * N, device="cuda")
    won, _ = xp.xp_tune_gemm(M, N, K, 1.0, a, "row", K, b, "col", K, 0.0, c, "row", N, ws, reps=3)
    off = xp.xp_describe_config(0, "bf16", won)
    for _ in range(2):                                       # from the table, then from the file
        assert _gemm(xp, "bf16", 0, M, N, K) == aligned and _gemm(xp, "bf16", 0, M, N, K, skew=1) == off
        xp.xp_tune_save(tmp_path / "t.txt")
        xp.xp_tune_clear()
        xp.xp_tune_load(tmp_path / "t.txt")
    # an entry that names the shape alone serves every alignment whose call its variant can run
    general = xp.xp_describe_config(0, "bf16", 0)
    (tmp_path / "old.txt").write_text(f"gemm0 t1 b1 m{M} n{N} k{K} a1 b1 | {general}\n")
    xp.xp_tune_clear()
    xp.xp_tune_load(tmp_path / "old.txt")
    assert _gemm(xp, "bf16", 0, M, N, K) == general and _gemm(xp, "bf16", 0, M, N, K, skew=1) == general
    # a name that has changed since
    (tmp_path / "old.txt").write_text("gemm0 t1 b1 m40 n16384 k520 a1 b1 | bf16 few rows x 8 to 32 rows, eight waves split k, through registers, mfma16\n")
    assert "few rows" not in _fresh(lambda: _gemm(xp, "bf16", 0, 40, 16384, 520))
    xp.xp_tune_load(tmp_path / "old.txt")
    assert "few rows" in _gemm(xp, "bf16", 0, 40, 16384, 520)
    xp.xp_tune_clear()
