"""The names behind the fitted times, and the arithmetic of time_variants.py; no GPU needed."""
import pathlib
import random
import re

import pytest

from paper_2505_02146_amd import time_variants as tv

CSRC = pathlib.Path(tv.__file__).parent / "csrc"


def test_fitted_rows_name_variants():
    """A row whose name matches no variant is left out of the comparison without a word."""
    from paper_2505_02146_amd import xp
    text = (CSRC / "xp_fitted_times.inc").read_text()
    tables = {t: re.findall(r'^    \{"([^"]+)"', text.split(t + "[] = {")[1].split("};")[0], flags=re.M) for t in ("kFitBf16", "kFitI8", "kFitConv")}
    for table, rows in tables.items():
        kind = "i8" if table == "kFitI8" else "bf16"
        names = {xp.xp_describe_config(xp.XP_OP_GEMM, kind, v) for v in range(xp.xp_num_configs(xp.XP_OP_GEMM, kind))}
        assert rows and len(set(rows)) == len(rows) and set(rows) <= names, set(rows) - names


@pytest.mark.parametrize("align", ["aligned", "any"])
@pytest.mark.parametrize("family", tv.FAMILIES)
def test_drawn_calls_fit_the_buffers(family, align):
    rng, again = random.Random(3), random.Random(3)
    for _ in range(200):
        c = tv.draw(rng, family, align)
        assert c == tv.draw(again, family, align)
        if family == "conv":
            p = (c["h"] + 2 * c["pad"] - c["r"]) // c["stride"] + 1
            sizes, extents = (c["n"] * c["h"] ** 2 * c["cin"], c["cout"] * c["r"] ** 2 * c["cin"], c["n"] * p * p * c["cout"]), (c["cin"],)
            unit = 32
        else:
            n = max(c["batch"], 1)
            sizes, extents = (n * c["M"] * c["K"], n * c["N"] * c["K"], n * c["M"] * c["N"]), (c["M"], c["N"], c["K"])
            unit = 16 if family.endswith("i8") else 8
        assert max(sizes[:2]) <= tv.MAX_OPERAND and sizes[2] <= tv.MAX_OUT and min(extents) >= 1
        assert align == "any" or all(e % unit == 0 for e in extents)


def test_summary_and_comparison():
    call = lambda m, chosen: dict(family="gemm_bf16", M=m, chosen=chosen, us={"a": 10.0, "b": 20.0})
    before, after = [call(1, "a"), call(2, "b"), call(3, "a")], [call(1, "b"), call(2, "a"), call(3, "a")]
    assert tv.summary(after)[0].startswith("gemm_bf16: 3 calls, the chosen variant over the best: geometric mean 1.260, 1 more than 5 % slower")
    assert tv.compare(before, after)[0] == "3 calls in both, 2 choices differ: 1 more than 5 % faster, 1 more than 5 % slower"
