"""Last decode pass above D = 2^24: a workgroup goes from sender to sender and from tile to tile with the next tile on its way.  Means against a plain float64
inverse transform of the dequantized payloads, and the additive calls, one sender at a time, leave the same sums."""
import pytest

from oracle import eden_oracle as o
from tests import parity

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


def _decoded(msg, d, seed, client, bits):
    """H D^-1 of one message of b = 1 or 4, on the GPU in float64."""
    m = o.Message.from_bytes(bytes(msg[:64].cpu().numpy()) + bytes(8 * ((1 << int(msg[4])) * bits // 64)))
    D = 1 << m.log2D
    if bits == 4:
        idx = torch.stack([msg[64:64 + D // 2] & 15, msg[64:64 + D // 2] >> 4], 1).view(-1).long()
    else:
        shifts = torch.arange(8, device="cuda", dtype=torch.uint8)
        idx = ((msg[64:64 + D // 8, None] >> shifts) & 1).view(-1).long()
    y = torch.tensor(o.tables(bits)[1], device="cuda")[idx] * (m.S / D ** 0.5)
    del idx
    for bit in range(m.log2D):
        pairs = y.view(-1, 2, 1 << bit)
        y = torch.stack([pairs[:, 0] + pairs[:, 1], pairs[:, 0] - pairs[:, 1]], 1).view(-1)
    signs = torch.from_numpy(o.rademacher(seed, client, D)[:d].astype("f4")).cuda()
    return y[:d] * signs


# tiles of 2^15 and 2^16 (two workgroups each), fewer and more of them than compute units, ragged ends inside a quad and a tile; one sender, several, and
# both kinds of workspace slots side by side; from nine senders of one bit on the tile goes through the LDS as a whole
@pytest.mark.parametrize("d,budgets", [((1 << 24) + 1, [1024]), ((1 << 25) - 70_003, [256, 256]), ((1 << 26) - 1, [1024, 256, 1024]), ((1 << 26) + 65_538, [256]),
                                       ((1 << 26) + 5, [256, 1024]), ((1 << 27) - 131_071, [1024]), ((1 << 24) + 1, [256] * 9), ((1 << 25) + 70_003, [256] * 10)])
def test_means_of_large_vectors(d, budgets):
    from paper_2108_08842_amd import eden
    n, seed = len(budgets), 17
    ctx = eden.Context(d_max=d, n_max=n, device=0)
    gen = torch.Generator(device="cuda").manual_seed(d)
    ids = list(range(3, 3 + n))
    msgs = ctx.encode([torch.randn(d, generator=gen, device="cuda") for _ in range(n)], ids, budgets, seed)
    mean = torch.full((d + 4,), 0.25, device="cuda")
    ctx.decode_mean(msgs, ids, budgets, d, seed, mean[:d])
    assert bool((mean[d:] == 0.25).all())
    acc = torch.zeros(d + 4, device="cuda")
    for c in range(n):
        ctx.decode_accumulate([msgs[c]], [ids[c]], [budgets[c]], d, seed, acc[:d])
    assert bool((acc[d:] == 0.0).all())
    ctx.finalize_mean(acc[:d], n)
    if 256 in budgets:                                           # scaled and added in one rounding by the one call, in two by the others
        assert float((acc[:d] - mean[:d]).norm() / mean[:d].norm()) <= 2.0 ** -23
    else:
        assert torch.equal(acc[:d], mean[:d])
    assert ctx.last_device_status() == 0
    ctx.close()
    want = torch.zeros(d, device="cuda", dtype=torch.float64)
    for c in range(n):
        want += _decoded(msgs[c], d, seed, ids[c], budgets[c] // 256)
    want /= n
    err = float((mean[:d].double() - want).norm() / want.norm())
    assert err <= parity.MEAN_REL_L2, err
