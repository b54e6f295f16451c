"""GPU parity of the time-segmented forward against the fp64 oracle, across decay rates.

Shapes with few (batch, channel) rows, which every test here asserts of its own, cut the sequence into time segments: a pass
computes each segment's aggregate (P, H) -- the product of abar over the segment
and the state reached from zero -- and the scan of segment s starts from h0 folded
with the aggregates of segments 0..s-1.  How much the fold carries depends on the
decay: with a very fast decay P underflows to zero and each segment starts from
the previous segment's last few timesteps alone; with the decay of the MambaByte
layers over long segments P is tiny; with a slow decay P stays near 1 and the
state of every earlier segment reaches the end of the sequence, so an error in
P would compound over the folds.  Waves whose channels mix fast and slow decay
are covered too.  Bars: 2e-3 on y, 1e-4 on h_last.
"""
import numpy as np
import pytest
import torch

from gpu_util import announce, check_against_oracle, gpu_fwd, has_gpu
from plan_util import plan
from paper_2401_13660_amd.inputs import make_inputs

pytestmark = [pytest.mark.gpu, pytest.mark.skipif(not has_gpu(), reason="needs a GPU")]


def _cut(shape, pieces=None):
    """The library cuts this shape into time segments (with so many pre-pass pieces each)."""
    p = plan(shape)
    assert p.nseg > 1 and pieces in (None, p.pieces), p


def _scaled_A(inp, per_channel):
    """A[d, n] = -(n + 1) * per_channel[d]."""
    n = np.arange(1, inp.dstate + 1, dtype=np.float32)
    inp.A = (-np.outer(np.asarray(per_channel, dtype=np.float32), n)).astype(np.float32)
    return inp


@pytest.mark.parametrize("with_h0", [False, True])
def test_fast_decay_stops_at_once(with_h0):
    # A = -500 (n + 1): abar underflows within a few timesteps
    _cut((1, 256, 16384), pieces=1)
    inp = _scaled_A(make_inputs(1, 256, 16384, 16, seed=41, with_h0=with_h0), [500.0] * 256)
    announce(f"segments, fast decay (1, 256, 16384), h0={with_h0}")
    y, h = gpu_fwd(inp)
    check_against_oracle(inp, y, h)


def test_layer_decay_long_segments():
    # (1, 1528, 20480): 191 chains, 5 segments of 4096 bytes in 4 pre-pass pieces each, the
    # layers' A = -(n + 1)
    _cut((1, 1528, 20480), pieces=4)
    inp = make_inputs(1, 1528, 20480, 16, seed=42, with_h0=True)
    announce("segments, layer decay (1, 1528, 20480)")
    y, h = gpu_fwd(inp)
    rows = np.arange(0, 1528, 5)
    check_against_oracle(inp, y, h, rows=rows)


@pytest.mark.parametrize("shape", [(1, 256, 16384), (1, 61, 4112)])
def test_slow_decay_reads_whole_segments(shape):
    # A = -1e-3 (n + 1): the product over a segment stays near 1, the carry of
    # every earlier segment reaches the end of the sequence
    nb, dim, L = shape
    _cut(shape)
    inp = _scaled_A(make_inputs(nb, dim, L, 16, seed=43, with_h0=True), [1e-3] * dim)
    announce(f"segments, slow decay {shape}")
    y, h = gpu_fwd(inp)
    check_against_oracle(inp, y, h)


def test_waves_mixing_fast_and_slow_decay():
    # channels alternate in blocks of 4: every 8-channel wave holds both kinds,
    # except that the last 16 channels are all fast
    dim = 80
    scale = [500.0 if (d // 4) % 2 == 0 else 1e-2 for d in range(dim)]
    scale[-16:] = [500.0] * 16
    _cut((2, dim, 8192))
    inp = _scaled_A(make_inputs(2, dim, 8192, 16, seed=44, with_h0=True), scale)
    announce("segments, mixed decay (2, 80, 8192)")
    y, h = gpu_fwd(inp)
    check_against_oracle(inp, y, h)


def test_segmented_equals_itself_with_h_last_on_h0():
    # the aggregate pass reads h0 for the copy it leaves in the carry; with h_last
    # written over h0 the result must not change (bit for bit)
    import paper_2401_13660_amd as mb
    from gpu_util import to_device
    _cut((1, 256, 16384))
    inp = make_inputs(1, 256, 16384, 16, seed=45, with_h0=True)
    announce("segments, h_last over h0 (1, 256, 16384)")
    y_ref, h_ref = gpu_fwd(inp)
    t = to_device(inp)
    state = t["h0"].clone()
    y, h = mb.scan_fwd(t["u"], t["delta"], t["A"], t["B"], t["C"], D=t["Dskip"], dt_bias=t["dt_bias"],
                       z=t["z"], h0=state, h_last=state)
    torch.cuda.synchronize()
    assert h.data_ptr() == state.data_ptr()
    assert torch.equal(y, y_ref) and torch.equal(state, h_ref)
