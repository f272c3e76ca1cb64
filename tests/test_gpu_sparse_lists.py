"""The m-of-64 budgets by lists of the kept coordinates (k_sparse_gather, k_sparse_scatter_list) against the kernels that test every coordinate against
masks: a few groups of 64 blocks are gathered by a team of waves, one sender's values scattered by masks.  The same values in the same
order of additions: equal to the last bit.  (A vector of up to half a group is scattered by masks whatever the number of senders; from 24 kept on, large
launches alone gather by lists.)"""
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


# whole groups of 4096 coordinates, one coordinate more and less, a ragged block; senders that do not fill the last turn of four; m at which a wave has one,
# two and three or four values per lane, and the first m that takes masks again; vectors on every alignment of four bytes
@pytest.mark.parametrize("d,n", [(2048, 8), (2049, 8), (300_007, 17), (73 * 4096, 15), (61 * 4096 + 1, 18), (511 * 4096 - 1, 3), (513 * 4096 + 65, 2), (520 * 4096 - 63, 5)])
@pytest.mark.parametrize("m", [1, 6, 8, 9, 16, 17, 63])
def test_lists_and_masks_agree(d, n, m):
    from paper_2108_08842_amd import eden
    b = eden.B_SPARSE(m)
    ctx = eden.Context(d_max=d, n_max=n, device=0)
    gen = torch.Generator(device="cuda").manual_seed(64 * d + m)
    flat = [torch.randn(d + 4, generator=gen, device="cuda") for _ in range(n)]
    xs = [f[c % 4:c % 4 + d] for c, f in enumerate(flat)]
    ids = list(range(7, 7 + n))
    msgs = ctx.encode(xs, ids, [b] * n, 99)
    for c in {0, 1, n - 1}:
        alone = ctx.encode([xs[c]], [ids[c]], [b], 99)[0]
        assert torch.equal(alone, msgs[c]), c
    mean = torch.full((d,), float("nan"), device="cuda")
    ctx.decode_mean(msgs, ids, [b] * n, d, 99, mean)
    acc = torch.zeros(d, device="cuda")
    for c in range(n):
        ctx.decode_accumulate([msgs[c]], [ids[c]], [b], d, 99, acc)
    ctx.finalize_mean(acc, n)
    assert torch.equal(mean, acc)
    # added to what is there: the sum of all senders first, then that to the old value, one fp32 addition for each call
    total = torch.zeros(d, device="cuda")
    ctx.decode_accumulate(msgs, ids, [b] * n, d, 99, total)
    ctx.finalize_mean(total.clone(), n, out=mean)
    assert torch.equal(mean, acc)
    one = torch.zeros(d, device="cuda")
    ctx.decode_accumulate(msgs[:1], ids[:1], [b], d, 99, one)
    more = torch.randn(d, generator=gen, device="cuda")
    want = more + total
    ctx.decode_accumulate(msgs, ids, [b] * n, d, 99, more)
    assert torch.equal(more, want)
    ctx.decode_accumulate(msgs[:1], ids[:1], [b], d, 99, more)
    assert torch.equal(more, want + one)
    ctx.decode_accumulate(msgs, ids, [b] * n, d, 99, more)
    assert torch.equal(more, (want + one) + total)
    assert ctx.last_device_status() == 0
    ctx.close()


# the two largest forms: more than 64 KiB of lists in the scatter (32 senders, 16 of 64 kept), and x beyond the size of the memory-side cache, which the gather
# reads with another policy (ragged end, vectors on every alignment; 47 of 64: lists in the launch of seven, masks in that of one)
@pytest.mark.parametrize("d,n,m", [(50_001, 32, 16), (10_000_001, 7, 6), (10_000_001, 7, 47)])
def test_the_largest_lists(d, n, m):
    test_lists_and_masks_agree(d, n, m)
