"""The block transfer that allocates nothing (its id lists sit in a static device array of the library)
against the ordinary one: same bits in the destination pool, on two calls in a row, the second smaller."""
import numpy as np
import pytest
import torch

from paper_2501_05460_amd import binding as B

pytestmark = pytest.mark.gpu

BT, DIM = 16, 96


def _pools(n_src, n_dst, seed):
    src = B.MMCache(n_src, BT, DIM, True)
    a, b = B.MMCache(n_dst, BT, DIM, True), B.MMCache(n_dst, BT, DIM, True)
    g = torch.Generator(device="cuda").manual_seed(seed)
    bits = torch.randint(-32768, 32767, (n_src, BT, DIM), dtype=torch.int16, device="cuda", generator=g)
    src.pool_tensor().view(torch.int16).copy_(bits)
    for c in (a, b):
        c.pool_tensor().view(torch.int16).fill_(-21555)
    return src, a, b


def test_noalloc_transfer_matches_the_ordinary_transfer_twice_in_a_row():
    src, a, b = _pools(300, 260, 7)
    src_ids = src.alloc(300 * BT)
    a_ids, b_ids = a.alloc(260 * BT), b.alloc(260 * BT)
    assert a_ids == b_ids
    rng = np.random.default_rng(5)
    # first call: 200 blocks in a scattered order; second call: 37 other blocks onto partly the same places
    for n, seed in ((200, 1), (37, 2)):
        pick_s = [src_ids[i] for i in rng.permutation(300)[:n]]
        pick_d = [a_ids[i] for i in rng.permutation(260)[:n]]
        src.transfer_to(pick_s, a, pick_d)
        src.transfer_to(pick_s, b, pick_d, noalloc=True)
        torch.cuda.synchronize()
        pa, pb = a.pool_tensor().view(torch.int16), b.pool_tensor().view(torch.int16)
        assert torch.equal(pa, pb), n
        # and both hold the source blocks (checked without the library: plain tensor indexing)
        want = src.pool_tensor().view(torch.int16)[torch.tensor(pick_s, device="cuda")]
        assert torch.equal(pb[torch.tensor(pick_d, device="cuda")], want), n
    untouched = b.pool_tensor().view(torch.int16) == -21555
    assert bool(untouched.any())          # blocks no call named still hold the fill value
    for c in (src, a, b):
        c.close()


def test_noalloc_transfer_of_lists_past_the_launch_arguments():
    """Lists of more than 896 blocks go through the static array: 2500, then 1900 scattered ids (the array still holds
    the first call's), then 896 of them, which ride in the launch arguments; against plain indexing."""
    n_src, n_dst = 2600, 2550
    src, a, b = _pools(n_src, n_dst, 11)
    a.close()
    src_ids, b_ids = np.array(src.alloc(n_src * BT)), np.array(b.alloc(n_dst * BT))
    want = torch.full((n_dst, BT, DIM), -21555, dtype=torch.int16, device="cuda")
    rng = np.random.default_rng(6)
    for n in (2500, 1900, 896):
        s, d = rng.permutation(src_ids)[:n], rng.permutation(b_ids)[:n]
        src.transfer_to(s.tolist(), b, d.tolist(), noalloc=True)
        torch.cuda.synchronize()
        want[torch.from_numpy(d).cuda()] = src.pool_tensor().view(torch.int16)[torch.from_numpy(s).cuda()]
        assert torch.equal(b.pool_tensor().view(torch.int16), want), n
    src.close()
    b.close()


@pytest.mark.parametrize("n", [896, 897])
def test_noalloc_transfer_on_both_sides_of_the_argument_limit(n):
    src, a, b = _pools(1000, 1000, 13)
    s, d = src.alloc(1000 * BT), a.alloc(1000 * BT)
    assert b.alloc(1000 * BT) == d
    rng = np.random.default_rng(n)
    pick_s, pick_d = [s[i] for i in rng.permutation(1000)[:n]], [d[i] for i in rng.permutation(1000)[:n]]
    src.transfer_to(pick_s, a, pick_d)
    src.transfer_to(pick_s, b, pick_d, noalloc=True)
    torch.cuda.synchronize()
    got = b.pool_tensor().view(torch.int16)
    assert torch.equal(got, a.pool_tensor().view(torch.int16))
    assert torch.equal(got[torch.tensor(pick_d, device="cuda")], src.pool_tensor().view(torch.int16)[torch.tensor(pick_s, device="cuda")])
    for c in (src, a, b):
        c.close()


def test_noalloc_transfer_rejects_what_it_cannot_hold_and_bad_ids():
    src, a, b = _pools(8, 8, 9)
    s_ids, b_ids = src.alloc(8 * BT), b.alloc(4 * BT)
    big = [0] * (65536 + 1)
    with pytest.raises(B.EpdError) as e:
        src.transfer_to(big, b, big, noalloc=True)
    assert e.value.status == B.EPD_ERR_UNSUPPORTED and "65536" in str(e.value)
    with pytest.raises(B.EpdError) as e:
        src.transfer_to(s_ids[:2], b, [b_ids[0], 7], noalloc=True)     # block 7 of b is not allocated
    assert e.value.status == B.EPD_ERR_OFFSETS
    src.transfer_to([], b, [], noalloc=True)                           # empty: no-op
    torch.cuda.synchronize()
    assert bool((b.pool_tensor().view(torch.int16) == -21555).all())
    for c in (src, a, b):
        c.close()
