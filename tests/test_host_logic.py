"""Host-side launch logic of the library, run on the CPU.

The library's own rules (csrc/fwd_plan.hpp) compiled into a small host program, on the 256
compute units of an MI355X.
"""
import pytest

from plan_util import have_compiler, plan, plans

pytestmark = pytest.mark.skipif(not have_compiler(), reason="needs a C++ compiler")

U32 = 2 ** 32 - 1        # HIP's limit on workgroups x threads along a grid dimension


# batch x ceil(dim / 8) chains round the bounds of a launch with 4, 2 and 1 waves each, at a
# length that takes 4, 2 or 1 wave where they fit
@pytest.mark.parametrize("L", [1, 33, 272])
@pytest.mark.parametrize("chains", [2 ** 24 - 1, 2 ** 24, 2 ** 25 - 1, 2 ** 25, 2 ** 26 - 4, 2 ** 26, 2 ** 28])
def test_every_problem_fits_its_launch(L, chains):
    p = plan((chains, 8, L))
    assert p.workgroups * p.threads <= U32, p
    if p.kernel == "ring":
        assert p.workgroups * (p.threads // 64) >= chains * p.waves
    else:
        assert p.kernel == "row" and p.workgroups * p.threads >= 8 * chains
    # one wave per chain fits below 2^26 chains; the row kernel takes a timestep or two of many
    assert (p.kernel == "ring") == (chains < 2 ** 26 and L > 1)
    assert plan((chains, 8, L), h0=True).kernel == ("ring" if chains < 2 ** 26 else "row")
    aligned16 = plan((1, 8 * chains, 16))
    assert aligned16.workgroups * aligned16.threads <= U32, aligned16


def _rule(chains: int, L: int):
    """segments, their length, pre-pass pieces."""
    n = 1
    if chains < 224 and L >= (2048 if chains <= 128 else 3072 if chains <= 160 else 4096 if chains < 192 else 16384):
        n = 1024 // chains if chains < 205 else 8
    if 256 < chains <= 288 and L >= 8192:
        n = 8
    n = min(n, L // 256, 128)
    if n <= 1:
        return 1, None, 1
    least = -(-L // n)
    m = 1
    if least >= 1024 and 2 * chains * (n - 1) <= 4096:
        m = 4 if least >= 3072 and 4 * chains * (n - 1) <= 4096 else 2
    seg = -(-least // (32 * m)) * (32 * m)
    return -(-L // seg), seg, m


def test_segments_follow_the_rule():
    shapes = [(1, 8 * c, L) for c in (1, 3, 8, 31, 100, 128, 129, 160, 161, 191, 192, 204, 205, 223, 224, 255, 256, 257, 264, 288, 289, 448,
                                      576, 1792)
              for L in (16, 256, 1008, 2047, 2048, 3071, 4095, 4096, 8190, 8192, 20480, 65536, 2 ** 24)]
    for (nb, dim, L), p in zip(shapes, plans(shapes, aligned=False)):
        n, seg, m = _rule(dim // 8, L)
        assert (p.nseg, p.pieces) == (n, m), (dim, L, p)
        assert (p.carry > 0) == (n > 1)
        if n > 1:
            assert p.seg_len == seg and seg % (32 * m) == 0 and seg >= 256
            assert (n - 1) * seg < L <= n * seg
    # worked by hand: segments, length, pieces
    hand = {(1, 8, 65536): (128, 512, 1), (1, 64, 2048): (8, 256, 1), (1, 512, 16384): (16, 1024, 2),
            (1, 1024, 32768): (8, 4096, 4), (1, 1528, 20480): (5, 4096, 4), (1, 1536, 16384): (5, 3328, 4), (1, 1528, 4095): (1, None, 1),
            (1, 2304, 8192): (8, 1024, 2), (1, 2304, 8191): (1, None, 1), (1, 2312, 8192): (1, None, 1), (2, 24, 8192): (32, 256, 1)}
    for (shape, want), p in zip(hand.items(), plans(list(hand), aligned=False)):
        assert (p.nseg, None if p.nseg == 1 else p.seg_len, p.pieces) == want, (shape, p)


def test_every_carry_fits_the_allocation_free_array():
    """On 256 compute units no carry exceeds the allocation-free call's 8 MiB."""
    shapes = [(1, 8 * c, L) for c in range(1, 400) for L in (2048, 4096, 8192, 16384, 20480, 32768, 65536, 2 ** 24)]
    for dtype in ("bf16", "f32"):
        assert 4 << 20 < max(p.carry for p in plans(shapes, dtype=dtype)) <= 8 << 20


def test_chunk_kernel_where_it_is_faster():
    """fp32 and, with checkpoints, bf16 problems of more than 256 MB whose chains are many, or few
    enough to be cut; whole slices in aligned rows only."""
    mb256 = 256 << 20

    def kernel(chains, nbytes, **kw):                    # the length that just passes, or not
        kw = {"dtype": "f32", **kw}
        per = (8 if kw["dtype"] == "bf16" else 16) + (4 if kw.get("ckpt") else 0) + (2 if kw["dtype"] == "bf16" else 0)
        L = (nbytes // (8 * chains * per * 16) + (nbytes > mb256)) * 16
        return plan((1, 8 * chains, L), **kw).kernel

    more, less = mb256 + 1, mb256
    for chains, want in {63: "ring", 64: "chunk", 223: "chunk", 224: "ring", 256: "ring", 257: "chunk", 307: "chunk",
                         308: "ring", 1791: "ring", 1792: "chunk", 28672: "chunk"}.items():
        assert kernel(chains, more) == want, chains
        assert kernel(chains, less) == "ring", chains
        assert kernel(chains, more, aligned=False) == "ring"
    assert [kernel(c, more, ckpt=True) for c in (1535, 1536)] == ["ring", "chunk"]
    bf = dict(dtype="bf16")
    assert plan((16, 3584, 512), **bf).kernel == "ring"
    assert [plan(s, ckpt=True, **bf).kernel for s in ((16, 3584, 512), (16, 3584, 320), (8, 3584, 2048))] == ["chunk", "ring", "ring"]
    assert plan((16, 3584, 1009), dtype="f32", aligned=True).kernel == "ring"
    segmented = plan((1, 1280, 65536), dtype="f32")
    assert segmented[:4] == ("chunk", 25, 2624, 1) and segmented.workgroups == 25 * 160 // 4


def test_row_kernel_for_a_few_timesteps_of_many_rows():
    """Without a first state or positions: bf16 up to 8 timesteps, from 16 chains per compute unit and 16 more per
    timestep; fp32 up to 4, from 8 and 24 more."""
    cu = 256
    for L in range(1, 12):
        for dtype, least in (("bf16", 16 + 16 * L if L <= 8 else None), ("f32", 8 + 24 * L if L <= 4 else None)):
            edge = (least or 1000) * cu
            below, at = plans([(edge - 1, 8, L), (edge, 8, L)], dtype=dtype)
            assert (below.kernel, at.kernel) == ("ring", "row" if least else "ring"), (L, dtype)
            if at.kernel == "row":
                assert at.workgroups * at.threads == 8 * edge and at.threads == 64 and at.nseg == 1
            for kw in (dict(h0=True), dict(npos=1)):
                assert plan((edge, 8, L), dtype=dtype, **kw).kernel == "ring"


def test_waves_per_chain():
    """8 up to one chain per compute unit, 4 above; fewer for short sequences of many chains;
    never more than there are slices of 16 timesteps."""
    want = {(256, 2048): 8, (257, 2048): 4, (256, 48): 2, (256, 33): 2, (256, 17): 2, (256, 9): 1,
            (768, 128): 4, (769, 128): 2, (769, 129): 4, (1024, 64): 2, (1024, 129): 4,
            (1025, 64): 1, (1025, 65): 2, (1025, 256): 2, (1025, 257): 4,
            (1791, 128): 2, (1792, 128): 1, (1792, 129): 2, (2048, 257): 4,
            (2049, 257): 2, (2049, 512): 2, (2049, 513): 4, (4096, 256): 2, (4097, 256): 1, (4097, 257): 2}
    got = plans([(1, 8 * c, L) for c, L in want], aligned=False)
    assert {k: p.waves for k, p in zip(want, got)} == want
