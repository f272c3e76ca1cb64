"""D = 2^25 .. 2^27: the kernel instances that serve rounds of one-bit and half-bit senders, pairs before the rotation, and rounds of
several budgets.  The reference is the method in float64 with torch on the GPU (the numpy oracle needs minutes for these sizes);
signs, sub-sampling and loss come from the library's hash streams, which other tests compare with the oracle's bit for bit."""
import math

import numpy as np
import pytest

from oracle import eden_oracle as o
from tests import parity

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")
Q1 = math.sqrt(2.0 / math.pi)


def _fwht64(u):
    """H u in place, Sylvester order, float64."""
    h = 1
    while h < u.numel():
        v = u.view(-1, 2, h)
        a = v[:, 0] + v[:, 1]
        v[:, 1].neg_().add_(v[:, 0])
        v[:, 0].copy_(a)
        h *= 2
    return u


def _bits(words, per, count):
    """The first `count` bits of little-endian words of `per` bits, as a bool tensor."""
    out = torch.empty((words.numel(), per), dtype=torch.bool, device=words.device)
    for k in range(per):
        out[:, k] = ((words >> k) & 1) != 0
    return out.view(-1)[:count]


def _signs(ctx, seed, client, D):
    return 1.0 - 2.0 * _bits(ctx.make_sign_bits(seed, client, D), 64, D).double()


def _header(msg):
    return [float(v) for v in msg[32:56].cpu().numpy().view(np.float64)]           # S, |x|^2, <R(x), Q>


def _check_one_bit_message(ctx, x64, msg, seed, client, b_q8, stats):
    """x64: the vector that is rotated, in float64.  Counts signs that differ from the exact ones (each within 1e-5 of zero) and
    compares |x|^2, <R(x), Q> and S; returns +1, -1 or 0 (not sent) per rotated coordinate as the message has it."""
    d = x64.numel()
    D = 1 << (d - 1).bit_length()
    z = torch.zeros(D, dtype=torch.float64, device="cuda")
    z[:d] = x64
    n2 = float((x64 * x64).sum())
    z = _fwht64(z.mul_(_signs(ctx, seed, client, D))).div_(math.sqrt(n2))
    if b_q8 == 128:
        pairs = torch.arange(D // 2, device="cuda")
        kept = 2 * pairs + _bits(ctx.make_subsample_bits(seed, client, D), 64, D // 2).long()
        sent = _bits(msg[64:], 8, D // 2)
        wrong, at = sent != (z[kept] >= 0), z[kept]
        q = torch.zeros(D, dtype=torch.int8, device="cuda")
        q[kept] = sent.to(torch.int8) * 2 - 1
    else:
        sent = _bits(msg[64:], 8, D)
        wrong, at = sent != (z >= 0), z
        q = sent.to(torch.int8) * 2 - 1
    assert float(at[wrong].abs().max()) <= parity.INDEX_BOUNDARY_TOL if wrong.any() else True
    parity._count(stats, 256, sent.numel(), int(wrong.sum()))
    S, N2, IP = _header(msg)
    assert abs(N2 - n2) <= 1e-12 * n2
    signs = z.sign() if b_q8 == 128 else q.double()              # the scale is over all coordinates, sent or not
    ip = math.sqrt(n2 / D) * Q1 * float((z * signs).sum())
    assert abs(IP - ip) <= parity.SCALE_RTOL * ip and abs(S - n2 / ip) <= parity.SCALE_RTOL * n2 / ip
    return q


def _decode_one_bit(ctx, q, msg, seed, client, bitmap):
    """x^ of one message in float64 (Sec. 2.2.2, 4.2), all D coordinates."""
    D = q.numel()
    y = q.double()
    if bitmap is not None:
        arrived = _bits(bitmap.view(torch.int32), 32, D // 1024)
        y = (y.view(-1, 1024) * arrived.double()[:, None]).view(-1)
    p = float((y != 0).sum()) / D
    return _fwht64(y).mul_(_signs(ctx, seed, client, D)).mul_(_header(msg)[0] * Q1 / p / math.sqrt(D))


def _vector(d, seed):
    g = torch.Generator(device="cuda").manual_seed(seed)
    x = torch.randn(d, generator=g, device="cuda")
    return x.mul_(torch.exp(2.0 * torch.rand(64, generator=g, device="cuda")).repeat_interleave((d + 63) // 64)[:d])


@pytest.mark.parametrize("d", [(1 << 24) + 40_001, (1 << 25) + 1, (1 << 26) - 70_001, (1 << 26) + 65_537, 1 << 27])
@pytest.mark.parametrize("budgets,drop", [([256, 256], 0.1), ([128, 128], 0.0), ([256, 128], 0.1)], ids=["one", "half", "one_and_half"])
def test_rounds_of_at_most_one_bit(d, budgets, drop):
    # the sign instances of the strided encode pass, the packed int16 first decode pass (integers up to 2^11 in fp16 slots) and the
    # 15- and 16-bit contiguous passes with fp16 slots alone; with loss, ragged last tiles and whole ones
    from paper_2108_08842_amd import eden
    D = 1 << (d - 1).bit_length()
    ids, seed = [11, 12], 9000 + d % 1000
    ctx = eden.Context(d_max=d, n_max=2, device=0)
    xs = [_vector(d, c) for c in ids]
    msgs = ctx.encode(xs, ids, budgets, seed)
    maps = [ctx.make_loss_bitmap(seed, ids[0], D, int(drop * 2 ** 32)), None] if drop else None
    print(f"d={d} budgets={budgets} drop={drop}", flush=True)
    stats = parity.EncodeParity()
    want = torch.zeros(d, dtype=torch.float64, device="cuda")
    for c in range(2):
        q = _check_one_bit_message(ctx, xs[c].double(), msgs[c], seed, ids[c], budgets[c], stats)
        want += _decode_one_bit(ctx, q, msgs[c], seed, ids[c], maps[c] if maps else None)[:d] / 2
    parity.finish_encode(stats)
    mean = torch.full((d,), float("nan"), device="cuda")
    ctx.decode_mean(msgs, ids, budgets, d, seed, mean, maps)
    assert float((mean.double() - want).norm() / want.norm()) <= parity.MEAN_REL_L2
    acc = torch.ones(d, device="cuda")
    ctx.decode_accumulate(msgs, ids, budgets, d, seed, acc, maps)
    assert float((acc.double() - 1.0 - 2.0 * want).norm() / (1.0 + 2.0 * want).norm()) <= parity.MEAN_REL_L2
    assert ctx.last_device_status() == 0 and ctx.last_decode_flags(2) == [0, 0]
    ctx.close()


@pytest.mark.parametrize("d,n", [((1 << 25) + 3, 2), (50_000_001, 1), ((1 << 26) + 77_777, 2), (1 << 27, 1)])
def test_pairs_before_the_rotation_above_two_to_the_25(d, n):
    # EDEN_B_HALF_PRE where the kept vector has 2^25 or 2^26 padded coordinates: gather and scatter of the 15-bit contiguous passes;
    # the mean and an accumulator that holds something, the last coordinate of an odd d among a pair
    from paper_2108_08842_amd import eden
    dk = (d + 1) // 2
    D = 1 << (dk - 1).bit_length()
    ids, budgets, seed = [3 + c for c in range(n)], [eden.B_HALF_PRE] * n, 77 + d % 1000
    ctx = eden.Context(d_max=d, n_max=n, device=0)
    xs = [_vector(d, 50 + c) for c in ids]
    msgs = ctx.encode(xs, ids, budgets, seed)
    print(f"pairs first: d={d} n={n}", flush=True)
    stats = parity.EncodeParity()
    want = torch.zeros(2 * dk, dtype=torch.float64, device="cuda")
    for c in range(n):
        src = 2 * torch.arange(dk, device="cuda") + _bits(ctx.make_subsample_bits(seed, ids[c], 2 * D), 64, dk).long()
        padded = torch.cat([xs[c].double(), torch.zeros(2 * dk - d, dtype=torch.float64, device="cuda")])
        q = _check_one_bit_message(ctx, 2.0 * padded[src], msgs[c], seed, ids[c], 256, stats)
        want[src] += _decode_one_bit(ctx, q, msgs[c], seed, ids[c], None)[:dk] / n
    parity.finish_encode(stats)
    want = want[:d]
    mean = torch.full((d,), float("nan"), device="cuda")
    ctx.decode_mean(msgs, ids, budgets, d, seed, mean)
    assert float((mean.double() - want).norm() / want.norm()) <= parity.MEAN_REL_L2
    acc = torch.ones(d, device="cuda")
    ctx.decode_accumulate(msgs, ids, budgets, d, seed, acc)
    assert float((acc.double() - 1.0 - n * want).norm() / (1.0 + n * want).norm()) <= parity.MEAN_REL_L2
    assert ctx.last_device_status() == 0
    ctx.close()


@pytest.mark.parametrize("d", [(1 << 24) + 100_003, (1 << 26) - 1, (1 << 26) + 300_001, (1 << 27) - 5])
def test_rounds_of_several_budgets_above_two_to_the_24(d):
    # one launch with every kind of sender: the shared instances of the strided passes, fp32 and fp16 slots in one contiguous pass.
    # A misplaced index, bit or row would show in two properties of every sender's reconstruction: <x^, x> = |x|^2 (Sec. 2.3), here to
    # 1e-5, and a squared error over all D coordinates of (1 / E q^2 - 1) |x|^2, of which the first d hold their share d / D at
    # least (the padding correlates the rotated coordinates) and all of it at most; the round is the mean of the senders decoded alone
    from paper_2108_08842_amd import eden
    D = 1 << (d - 1).bit_length()
    budgets = [256, eden.B_COIN(1.3), 1024, 128, 640, 2048, eden.B_COIN(3.7), eden.B_GRID(0.5224)]
    n = len(budgets)
    ids, seed = [20 + c for c in range(n)], 400 + d % 1000
    print(f"several budgets: d={d}", flush=True)
    ctx = eden.Context(d_max=d, n_max=n, device=0)
    xs = [_vector(d, 80 + c % 2) for c in range(n)]
    msgs = ctx.encode(xs, ids, budgets, seed)
    mean, alone = torch.full((d,), float("nan"), device="cuda"), torch.empty(d, device="cuda")
    ctx.decode_mean(msgs, ids, budgets, d, seed, mean)
    total = torch.zeros(d, dtype=torch.float64, device="cuda")

    def kept_energy(b):                                          # E q^2 of the quantizer on N(0, 1)
        if o.grid_delta(b):
            t = np.arange(-127, 128) * o.grid_delta(b)
            edges = np.concatenate([[-np.inf], (t[1:] + t[:-1]) / 2, [np.inf]])
            cdf = np.array([0.5 * (1 + math.erf(e / math.sqrt(2))) for e in edges])
            c = o.grid_centroids(o.grid_delta(b))
            return float(np.sum(np.diff(cdf) * np.concatenate([c[:0:-1], c]) ** 2))
        if b >= 0x40000:
            f = ((b & 0xFFFF) % 256) / 256
            k = (b & 0xFFFF) >> 8
            return (1 - f) * o.expected_q2(*o.tables(k)) + f * o.expected_q2(*o.tables(k + 1))
        if b % 256 == 128 and b > 256:
            return (o.expected_q2(*o.tables(b >> 8)) + o.expected_q2(*o.tables((b >> 8) + 1))) / 2
        return o.expected_q2(*o.tables(max(1, b >> 8)))

    for c in range(n):
        ctx.decode_mean(msgs[c:c + 1], ids[c:c + 1], budgets[c:c + 1], d, seed, alone)
        x64, a64 = xs[c].double(), alone.double()
        total += a64 / n
        n2 = float(x64.dot(x64))
        assert abs(_header(msgs[c])[1] - n2) <= 1e-12 * n2
        err = float((a64 - x64).dot(a64 - x64)) / n2
        full = 2.0 / Q1 ** 2 - 1.0 if budgets[c] == 128 else 1.0 / kept_energy(budgets[c]) - 1.0
        assert 0.98 * full * d / D < err < 1.02 * full, (c, budgets[c], err, full)
        if budgets[c] != 128:                                    # (half of its coordinates do not travel: unbiased, not tangent)
            assert abs(float(x64.dot(a64)) / n2 - 1.0) < 1e-5, (c, budgets[c])
    assert float((mean.double() - total).norm() / total.norm()) <= 1e-6          # fp32 sums of the same values in another grouping
    assert ctx.last_device_status() == 0
    ctx.close()
