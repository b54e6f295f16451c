"""GPU parity of the forward scan at the edges of its time slices, against the fp64 oracle.

The forward deals 16-timestep slices of 8 channels round 1 to 8 waves of a workgroup,
runs up to 15 timesteps after the last full slice one by one, and takes rows that start at
any element.  The shapes below put the sequence's end on either side of a slice, a round of
slices and a time segment, leave channels over, and choose each number of waves per chain:
by the slices (up to 4), by few chains (8), by thousands of chains (1).  Bars: 2e-3 on y
(fp32 arithmetic; observed below 1e-5), 1e-4 on states.
"""
import numpy as np
import pytest
import torch

import oracle
from gpu_util import announce, check_against_oracle, gpu_fwd, has_gpu, to_device
from paper_2401_13660_amd.inputs import make_inputs
from parity import TOL_H, TOL_Y, TOL_Y_BF16_OUT, rel_err

pytestmark = [pytest.mark.gpu, pytest.mark.skipif(not has_gpu(), reason="needs a GPU")]


@pytest.mark.parametrize("dtype", ["bf16", "f32"])
@pytest.mark.parametrize("L", [1, 2, 15, 17, 31, 32, 33, 49, 63, 64, 65, 127, 128, 129, 255, 257])
def test_lengths_round_the_slices(L, dtype):
    inp = make_inputs(2, 13, L, 16, dtype=dtype, seed=300 + L, with_h0=True, gated=L % 2 == 1)
    announce(f"ring L={L} {dtype}")
    y, h = gpu_fwd(inp)
    check_against_oracle(inp, y, h)


@pytest.mark.parametrize("shape", [
    (1, 8, 1000),            # one chain, 8 waves
    (3, 1024, 70),           # 384 chains: 4 waves each, a short slice after 4
    (2, 2048, 263),          # 512 chains, 16 full slices and 7 timesteps
    (32, 1030, 51),          # 4,128 chains of 4 slices: one wave each, dead lanes
    (1, 40, 4301),           # 5 chains: time segments, the last one of odd length
    (6, 2048, 135),          # 1,536 chains of 8 slices: 2 waves each
])
def test_waves_per_chain_and_segments(shape):
    nb, dim, L = shape
    inp = make_inputs(nb, dim, L, 16, seed=77, with_h0=True, A_kind="random")
    announce(f"ring {shape}")
    rows = np.unique(np.concatenate([np.arange(0, nb * dim, max(1, nb * dim // 300)), [nb * dim - 1]]))
    y, h = gpu_fwd(inp, out_dtype=torch.bfloat16)
    check_against_oracle(inp, y, h, rows=rows, tol_y=TOL_Y_BF16_OUT)


@pytest.mark.parametrize("dtype,L", [("bf16", 96), ("bf16", 101), ("f32", 101), ("f32", 704)])
def test_rows_at_any_element(dtype, L):
    """Every activation and y one element past an aligned address: the same results."""
    import paper_2401_13660_amd as mb
    inp = make_inputs(2, 9, L, 16, dtype=dtype, seed=5, with_h0=True)
    t = to_device(inp)

    def shifted(x):
        buf = torch.empty(x.numel() + 1, dtype=x.dtype, device=x.device)
        buf[1:] = x.reshape(-1)
        return buf[1:].view(x.shape)

    s = {k: shifted(t[k]) for k in ("u", "delta", "z", "B", "C")}
    out = shifted(torch.zeros((2, 9, L), device="cuda:0"))
    announce(f"ring unaligned {dtype} L={L}")
    y, h = mb.scan_fwd(s["u"], s["delta"], t["A"], s["B"], s["C"], D=t["Dskip"], dt_bias=t["dt_bias"], z=s["z"],
                       h0=t["h0"], out=out, return_last_state=True)
    torch.cuda.synchronize()
    y_ref, h_ref = oracle.scan_inputs(inp)
    assert rel_err(y.cpu().numpy(), y_ref) <= TOL_Y
    assert rel_err(h.cpu().numpy(), h_ref) <= TOL_H


@pytest.mark.parametrize("L", [9, 40, 75, 3301])
def test_positions_in_every_part(L):
    """States in full slices, in the timesteps after them and before the first; y and h_last
    are those of the plain call bit for bit, with h_last written over h0."""
    import paper_2401_13660_amd as mb
    inp = make_inputs(2, 11, L, 16, seed=8, with_h0=True)
    pos = np.array([[-1, 0], [7, L // 2], [L - 1, L - 2], [min(15, L - 1), min(16, L - 1)], [L, -2]], dtype=np.int32)
    t = to_device(inp)
    args = (t["u"], t["delta"], t["A"], t["B"], t["C"])
    kw = dict(D=t["Dskip"], dt_bias=t["dt_bias"], z=t["z"])
    announce(f"ring positions L={L}")
    y0, h0_last = mb.scan_fwd(*args, h0=t["h0"], return_last_state=True, **kw)
    state = t["h0"].clone()
    y, h, h_at = mb.scan_fwd(*args, h0=state, h_last=state, positions=torch.from_numpy(pos).to("cuda:0"), **kw)
    torch.cuda.synchronize()
    assert torch.equal(y, y0) and torch.equal(h, h0_last)
    _, _, ref = oracle.scan_inputs(inp, positions=pos)
    got = h_at.cpu().numpy()
    assert np.isnan(got[4]).all()
    assert rel_err(got[:4], ref[:4]) <= TOL_H
    assert np.array_equal(got[2, 0], h0_last[0].cpu().numpy())


@pytest.mark.parametrize("L", [7, 16, 83, 4099])
def test_more_positions_than_lanes(L):
    """130 positions per batch element, valid ones, -1 and ones past both ends among the first
    64, the second and the last 2: all looked for 64 at a time by the ring kernel (and by the
    16-timestep kernel at L = 16), in full slices, in the timesteps after them, in segments."""
    import paper_2401_13660_amd as mb
    from test_gpu_positions import check_states
    inp = make_inputs(2, 11, L, 16, seed=9, with_h0=True)
    rng = np.random.default_rng(L)
    pos = rng.integers(0, L, (130, 2)).astype(np.int32)
    for k in (0, 63, 64, 127, 128, 129):
        pos[k] = rng.permutation([L - 1, -1])
    for k, p in ((5, L), (62, -2), (65, -2), (100, 2 ** 31 - 1), (126, -2 ** 31)):
        pos[k, k % 2] = p
    t = to_device(inp)
    announce(f"ring, 130 positions, L={L}")
    _, h, h_at = mb.scan_fwd(t["u"], t["delta"], t["A"], t["B"], t["C"], D=t["Dskip"], dt_bias=t["dt_bias"], z=t["z"],
                             h0=t["h0"], positions=torch.from_numpy(pos).to("cuda:0"), return_last_state=True)
    torch.cuda.synchronize()
    check_states(inp, pos, h_at, h)
