"""The quantizers that search in lane masks (b = 3, k + 1/2, the general non-integer budgets, launches of different budgets) against those of the
launches of one b = 1, 2 or 4: the rotated values are the same, so a coordinate quantized with I_k has the index that it has in the message of b = k,
whatever the budget and the launch.  No index may differ: every compare is against the same threshold."""
import numpy as np
import pytest

from oracle import eden_oracle as o
from tests import parity

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


def _indices(msg, seed):
    m = parity.to_oracle_message(msg)
    D = 1 << m.log2D
    if o.mixed(m.b_q8):
        up = o.upgraded_mask(seed, m.client, D)
        return o.unpack_mixed(m.payload, D, m.b_q8, up), up
    if o.fractional(m.b_q8):
        up = o.coin_bits(seed, m.client, D, m.b_q8 & 0xFF)
        return o.unpack_fractional(m.payload, D, m.b_q8, up), up
    bits, _ = o.budget(m.b_q8)
    return o.unpack_indices(m.payload[:D * bits // 32], bits, D), None


# wave tiles of the strided pass from its shortest to its longest (a wave has one row to many), workgroup tiles of 7 to 10 bits; values of every level;
# |x| beyond 1.4e38, where the outer thresholds are infinite
@pytest.mark.parametrize("d", [4097, 9000, 70_000, 200_000, 500_001, (1 << 20) - 1, (1 << 21) - 3, 3_000_001, (1 << 22) + 1, (1 << 23) + 1])
@pytest.mark.parametrize("spiked", [False, True])
def test_an_index_does_not_depend_on_the_budget_beside_it(d, spiked):
    from paper_2108_08842_amd import eden
    seed, client = 91, 12
    rng = np.random.default_rng(d)
    x = rng.standard_normal(d)
    if spiked:                                                   # (the transform stays below the largest float: sum |x| <= 3.3e38)
        x *= 0.04e38 / np.abs(x).sum()
        x[rng.choice(d, 3, replace=False)] = 1.08e38 * rng.choice([-1.0, 1.0], 3)
    x = torch.from_numpy(x.astype(np.float32)).cuda()
    budgets = [256, 512, 768, 1024, 384, 640, 896] + [eden.B_COIN(b) for b in (1.3, 1.9, 2.2, 2.7, 3.1, 3.8)]
    ctx = eden.Context(d_max=d, n_max=len(budgets), device=0)
    alone = {b: _indices(ctx.encode([x], [client], [b], seed)[0], seed) for b in budgets}
    beside = ctx.encode([x] * len(budgets), [client] * len(budgets), budgets, seed)
    assert ctx.last_device_status() == 0
    for b, msg in zip(budgets, beside):
        idx, up = _indices(msg, seed)
        assert np.array_equal(idx, alone[b][0]), b
        k, _ = o.budget(b)
        low = idx if up is None else idx[~up]
        assert low.max() < 1 << k and np.unique(low).size >= (2 if spiked else 1 << k), b
        if up is not None:
            assert np.array_equal(low, alone[256 * k][0][~up]), b
            assert np.array_equal(idx[up], alone[256 * (k + 1)][0][up]), b
    ctx.close()


# the guess of b = 4 multiplies values and thresholds by a power of two where the outermost threshold is below 2^-60 or above 2^60: a vector times a power of
# two has the same indices, and <R(x), Q> times that power, at both sides of both lines (the threshold is 2.4 |x|: here 2^11 to 2^13 times the factor)
@pytest.mark.parametrize("d", [300_007, (1 << 21) - 3, (1 << 23) + 1])
def test_four_bits_of_a_scaled_vector(d):
    from paper_2108_08842_amd import eden
    gen = torch.Generator(device="cuda").manual_seed(d)
    x = torch.randn(d, generator=gen, device="cuda")
    x = torch.where(x.abs() < 2.0 ** -20, x.sign() * 2.0 ** -20, x)    # (no factor makes a subnormal)
    ctx = eden.Context(d_max=d, n_max=1, device=0)
    want = parity.to_oracle_message(ctx.encode([x], [3], [1024], 5)[0])
    for k in (-100, -74, -72, -71, 46, 47, 48, 50, 100):
        got = parity.to_oracle_message(ctx.encode([x * 2.0 ** k], [3], [1024], 5)[0])
        assert np.array_equal(got.payload, want.payload) and got.IP == want.IP * 2.0 ** k and got.N2 == want.N2 * 4.0 ** k, k
    assert ctx.last_device_status() == 0
    ctx.close()
