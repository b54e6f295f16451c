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
    m = 2 if n <= 16 and 2 * chains * (n - 1) <= 1024 else 1
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
    hand = {(1, 8, 65536): (128, 512, 1), (1, 64, 2048): (8, 256, 2), (1, 584, 2048): (8, 256, 2), (1, 592, 2048): (8, 256, 1), (1, 80, 4352): (17, 256, 1), (1, 512, 16384): (16, 1024, 2),
            (1, 1024, 32768): (8, 4096, 4), (1, 1528, 20480): (5, 4096, 4), (1, 1536, 16384): (5, 3328, 4), (1, 1528, 4095): (1, None, 1),
            (1, 2304, 8192): (8, 1024, 2), (1, 2304, 8191): (1, None, 1), (1, 2312, 8192): (1, None, 1), (2, 24, 8192): (32, 256, 1)}
    for (shape, want), p in zip(hand.items(), plans(list(hand), aligned=False)):
        assert (p.nseg, None if p.nseg == 1 else p.seg_len, p.pieces) == want, (shape, p)


def test_every_carry_fits_the_allocation_free_array():
    """On 256 compute units no carry exceeds the allocation-free call's 8 MiB."""
    shapes = [(1, 8 * c, L) for c in range(1, 1025) for L in (2048, 4096, 8192, 16384, 20480, 32768, 65536, 2 ** 24)]
    for dtype in ("bf16", "f32"):
        assert 4 << 20 < max(p.carry for p in plans(shapes, dtype=dtype)) <= 8 << 20


def _kernel(chains, mib, odd=False, **kw):
    """The kernel of the shortest sequence in whole lines (or an odd number of slices) of more than `mib` MiB."""
    kw = {"dtype": "f32", "out_bytes": 4, **kw}
    per = 3 * (4 if kw["dtype"] == "f32" else 2) + kw["out_bytes"] + (4 if kw.get("ckpt") else 0)
    L = ((mib << 20) // (8 * chains * per * 32) + 1) * 32
    return plan((1, 8 * chains, L - 16 if odd else L), **kw).kernel


def _chunk_ranges(mib, last, **kw):
    """The ranges of chains that the chunk kernel takes, first and last of each."""
    found, prev = [], False
    for c in range(1, last + 2):
        now = c <= last and _kernel(c, mib, **kw) == "chunk"
        if now and not prev:
            found.append([c])
        if prev and not now:
            found[-1].append(c - 1)
        prev = now
    return [tuple(f) for f in found]


# 256 compute units; (mib + 32, odd) rather than mib where an odd number of slices would fall below it
@pytest.mark.parametrize("want,mib,kw", [
    ([(64, 223), (257, 307), (1537, 1700)], 256, {}),
    ([(64, 223), (257, 307), (1537, 1700)], 320, dict(odd=True)),
    ([(64, 223), (257, 307), (1537, 1700)], 256, dict(npos=1)),
    ([(64, 223), (257, 307)], 256, dict(npos=40)),
    ([(32, 223), (257, 307)], 768, {}),
    ([(64, 223), (257, 307), (769, 1024), (1281, 1700)], 320, dict(ckpt=True)),
    ([(64, 223), (257, 307), (769, 1024), (1537, 1700)], 400, dict(ckpt=True, odd=True)),
    ([], 256, dict(dtype="bf16")),
    ([], 768, dict(dtype="bf16", ckpt=True)),
    ([], 320, dict(aligned=False, ckpt=True)),
])
def test_chunk_kernel_where_it_is_faster(want, mib, kw):
    last = 1700 if any(hi == 1700 for _, hi in want) else 700
    assert _chunk_ranges(mib, last, **kw) == want


def test_chunk_kernel_where_chains_fill_the_chip():
    """fp32 of any size from 192 timesteps where rounds of 2,048 chains are 7/8 full; bf16 with checkpoints
    where rounds of 1,024 are, and from 4,097 chains; nothing else below 256 MB."""
    f32 = dict(dtype="f32")
    for chains, want in {1791: "ring", 1792: "chunk", 2048: "chunk", 2049: "ring", 3583: "ring", 3584: "chunk", 4096: "chunk",
                         4097: "ring"}.items():
        assert plan((1, 8 * chains, 192), **f32).kernel == want, chains
        assert plan((1, 8 * chains, 192), ckpt=True, **f32).kernel == want, chains
        for other in (dict(dtype="f32", npos=1), dict(dtype="f32", aligned=False), dict(dtype="bf16", ckpt=True)):
            assert plan((1, 8 * chains, 192), **other).kernel == "ring"
        assert {plan((1, 8 * chains, L), **f32).kernel for L in (160, 200, 208)} == {"ring"}
    ck = dict(dtype="bf16", ckpt=True)
    for c, f32_out, bf16_out in ((1024, "ring", "ring"), (1791, "ring", "ring"), (1792, "chunk", "ring"), (1919, "chunk", "ring"),
                                 (1920, "chunk", "chunk"), (2048, "chunk", "chunk"), (2049, "ring", "ring"), (2687, "ring", "ring"),
                                 (2688, "chunk", "ring"), (2880, "chunk", "chunk"), (3073, "ring", "ring"), (4096, "chunk", "chunk"),
                                 (4097, "chunk", "chunk"), (8000, "chunk", "chunk")):
        assert (_kernel(c, 256, **ck), _kernel(c, 256, out_bytes=2, **ck)) == (f32_out, bf16_out), c
        assert _kernel(c, 256, dtype="bf16") == "ring"
        assert c > 4097 or _kernel(c, 200, **ck) == "ring"
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


def test_recording_changes_no_cut():
    """mb_scan_fwd_states and mb_scan_fwd_ckpt give mb_scan_fwd's bits: the ring and the chunk kernel may
    stand in for each other where neither cuts the sequence, the row kernel too for sequences of less than a
    slice; any two plans that cut must be alike."""
    shapes = [(1, 8 * c, L) for c in (1, 8, 31, 33, 63, 64, 100, 200, 223, 224, 256, 257, 288, 300, 307, 341, 358, 400, 513, 576, 700, 768,
                                      769, 1024, 1400, 2048, 3000, 4096, 5000)
              for L in (1, 4, 48, 512, 2048, 4096, 8192, 16384, 32768, 65536, 131072, 2 ** 20)]
    shapes += [(65536, 8, L) for L in (1, 2, 3, 4, 8, 9)]
    for dtype in ("bf16", "f32"):
        for out_bytes in (2, 4):
            kw = dict(dtype=dtype, out_bytes=out_bytes)
            plain = plans(shapes, **kw)
            for other in (plans(shapes, npos=1, **kw), plans(shapes, npos=40, **kw), plans(shapes, ckpt=True, **kw)):
                for shape, p, o in zip(shapes, plain, other):
                    if o.kernel != p.kernel:
                        assert {p.kernel, o.kernel} == {"ring", "chunk" if shape[2] >= 16 else "row"}, (shape, p, o)
                    assert p[1:4] == o[1:4], (shape, p, o)
                    assert p.nseg == 1 or p.kernel == o.kernel, (shape, p, o)
    assert {p.kernel for p in plain} == {"row", "ring", "chunk"}


def test_waves_per_chain():
    """8 up to one chain per compute unit, 4 above; fewer for short sequences of many chains;
    never more than there are slices of 16 timesteps."""
    want = {(256, 2048): 8, (257, 2048): 4, (256, 48): 2, (256, 33): 2, (256, 17): 2, (256, 9): 1,
            (768, 128): 4, (769, 128): 2, (769, 129): 4, (1024, 64): 2, (1024, 129): 4,
            (1025, 64): 1, (1025, 65): 2, (1025, 256): 2, (1025, 257): 4,
            (1791, 128): 2, (1792, 128): 1, (1792, 129): 2, (2048, 257): 4,
            (2816, 257): 4, (2817, 257): 2, (2817, 512): 2, (2817, 513): 4, (6144, 256): 2, (6145, 256): 1, (6145, 257): 2}
    got = plans([(1, 8 * c, L) for c, L in want], aligned=False)
    assert {k: p.waves for k, p in zip(want, got)} == want
