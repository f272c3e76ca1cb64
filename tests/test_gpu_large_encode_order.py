"""Encode above D = 2^24: the contiguous pass over 15 or 16 bits goes through the LDS in pieces and, at D = 2^27, through tile after tile in one
workgroup.  Every byte against plain fp32 butterflies in the order of the stages (the order is part of a message), and a message does not
depend on the senders beside it, header and all."""
import numpy as np
import pytest

from oracle import eden_oracle as o

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


def _stages(log2D):
    contiguous = [15] * (log2D == 27) + [*range(10, 15), *range(5, 10), *range(0, 5)]
    return contiguous + [*range(log2D - 6, log2D), *range(len(contiguous), log2D - 6)]


def _transformed(x, seed, client, log2D):
    """H (s o pad(x)) in fp32."""
    u = torch.zeros(1 << log2D, device="cuda")
    u[:x.numel()] = x
    u = u * torch.from_numpy(o.rademacher(seed, client, 1 << log2D).astype(np.float32)).cuda() + 0.0
    for bit in _stages(log2D):
        pairs = u.view(-1, 2, 1 << bit)
        u = torch.stack([pairs[:, 0] + pairs[:, 1], pairs[:, 0] - pairs[:, 1]], 1).view(-1)
    return u


# the smallest of a dimension and ragged ends of a tile at 2^25, 2^26 and 2^27 (one coordinate of a tile, all but some of one); several
# senders, so that a workgroup of the largest size goes on from one to the next.  No byte may differ: the operations are the same.
@pytest.mark.parametrize("d,n", [((1 << 24) + 1, 2), ((1 << 25) - 3, 1), ((1 << 26) - 70_001, 2), ((1 << 26) + 1, 3), ((1 << 27) - 65_537, 1), (1 << 27, 2)])
@pytest.mark.parametrize("bits", [2, 4])
def test_bytes_are_those_of_plain_butterflies_in_the_same_order(d, n, bits):
    from paper_2108_08842_amd import eden
    log2D = (d - 1).bit_length()
    ctx = eden.Context(d_max=d, n_max=n, device=0)
    half = 1 << (bits - 1)
    edges = torch.tensor(eden.get_tables(bits)[0], dtype=torch.float64, device="cuda")[half:]
    gen = torch.Generator(device="cuda").manual_seed(d)
    xs = [torch.randn(d, generator=gen, device="cuda") for _ in range(n)]
    ids = [3 + c for c in range(n)]
    msgs = ctx.encode(xs, ids, [256 * bits] * n, 77)
    alone = ctx.encode([xs[-1]], [ids[-1]], [256 * bits], 77)[0]
    assert torch.equal(alone, msgs[-1])
    for x, client, msg in zip(xs, ids, msgs):
        thr = (edges * torch.sqrt((x.double() ** 2).sum())).float()
        u = _transformed(x, 77, client, log2D)
        mag = torch.searchsorted(thr, u.abs()).to(torch.uint8)   # thresholds below |u|
        code = torch.where(torch.signbit(u), half - 1 - mag, half + mag).view(-1, 8 // bits)
        want = code[:, 0].clone()
        for k in range(1, 8 // bits):
            want |= code[:, k] << (bits * k)
        assert int((msg[64:64 + want.numel()] != want).sum()) == 0, client
        del u, mag, code, want
    assert ctx.last_device_status() == 0
    ctx.close()
