"""Attention of a few queries, whose waves share out the keys: edges of tiles, of shares and of the two workgroup sizes."""
import numpy as np
import pytest

from paper_2505_02146_amd import inputs
from tests.helpers import dev
from tests.test_gpu_attention import TIGHT, _gate, _run, xp  # noqa: F401

pytestmark = pytest.mark.gpu

# (batch, Lq, Lk): fewer keys than the waves share out; from 256 (head size 128) and 320 (64) on waves without a tile, one and
# several tiles a wave, a ragged last tile (of one key), all 16 queries; 256 problems and more, 448 (four waves) and more
CASES = [(1, 1, 64), (2, 16, 65), (3, 2, 256), (2, 1, 257), (2, 5, 319), (1, 16, 320), (2, 2, 321), (3, 1, 512), (2, 8, 513), (2, 15, 1000),
         (1, 3, 2049), (256, 1, 400), (257, 1, 600), (447, 1, 300), (448, 1, 257), (450, 2, 97), (450, 3, 520)]


@pytest.mark.parametrize("d,variant", [(64, 2), (128, 4)])
@pytest.mark.parametrize("scale", [0.125, -0.2])
def test_few_queries(xp, oracle, d, variant, scale):  # noqa: F811
    for n, (batch, Lq, Lk) in enumerate(CASES):
        got, ref, used, _ = _run(xp, oracle, batch=batch, Lq=Lq, Lk=Lk, d=d, dv=d, scale=scale, variant=variant, pad=((n % 2) * 8, 0, 8, 4),
                                 gap=n % 3 * 8, seed=n)
        assert used == variant
        _gate(got, ref, f"{batch} x {Lq} x {Lk} x {d}", TIGHT[variant])


@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("low", [range(0, 300), range(700, 1000), range(1, 1000)])
def test_shares_that_count_for_nothing(xp, d, low):  # noqa: F811
    """Keys whose scores are minus infinity, whole waves' shares of them, beside ordinary ones."""
    import torch
    batch, Lq, Lk = 2, 2, 1000
    Q, K, V = (inputs.normal((batch, L, d), 5, t).astype(np.float32) for L, t in ((Lq, 1), (Lk, 2), (Lk, 3)))
    Q[:, :, 0] = 1.0
    K[:, list(low), 0] = -np.inf
    bits = [inputs.to_bf16_bits(x) for x in (Q, K, V)]
    q, k, v = (torch.from_numpy(inputs.bf16_bits_to_f32(x)).double() for x in bits)
    ref = torch.matmul(torch.softmax(torch.matmul(q, k.transpose(1, 2).contiguous()) * 0.125, -1), v)
    o = torch.full((batch, Lq, d), 7.0, device="cuda")
    xp.xp_force_config(xp.XP_OP_ATTENTION, "bf16", -1)
    xp.xp_attention(batch, Lq, Lk, d, d, 0.125, dev(bits[0]), d, Lq * d, dev(bits[1]), d, Lk * d, dev(bits[2]), d, Lk * d, o, d, Lq * d,
                    q_type="bf16", k_type="bf16", v_type="bf16")
    # rounding the probabilities to bf16 moves each by 2^-9 at most, and the sum of them alike
    assert (o.cpu().double() - ref).norm() <= 2.0 ** -8 * ref.norm()


@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("scale", [0.125, -0.2])
@pytest.mark.parametrize("Lq", [1, 16])
def test_a_query_gets_the_same_result_among_few_and_among_many(xp, d, scale, Lq):  # noqa: F811
    """17 queries take the kernel that walks all keys with one reference maximum.  Rounded to bf16 against the same
    reference, the probabilities are the same ones; what differs is the order of fp32 sums over 1500 keys, 2^-24 sqrt(1500)
    = 2.3e-6 of the result and as much for the quotient's sum, taken four times (against other references: 2e-3)."""
    import torch
    batch, Lk = 3, 1500
    Q, K, V = (inputs.to_bf16_bits(inputs.normal((batch, L, d), 7, t)) for L, t in ((17, 1), (Lk, 2), (Lk, 3)))
    q, k, v = (dev(x.reshape(-1)) for x in (Q, K, V))
    xp.xp_force_config(xp.XP_OP_ATTENTION, "bf16", -1)

    def call(n):
        o = torch.full((batch, n, d), float("nan"), device="cuda")
        xp.xp_attention(batch, n, Lk, d, d, scale * d ** -0.5 * 8, q, d, 17 * d, k, d, Lk * d, v, d, Lk * d, o, d, n * d,
                        q_type="bf16", k_type="bf16", v_type="bf16")
        return o.double()
    few, many = call(Lq), call(17)[:, :Lq]
    assert (few - many).norm() <= 2e-5 * many.norm()
