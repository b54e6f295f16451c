"""The forward's chunk kernel: what it computes is what the ring kernel computes, bit for bit.

The chunk kernel takes problems of many chains of 8 channels, or of few enough to be cut into time
segments, most of them of more than 256 MB.  Uncut, its states and outputs come from the ring
kernel's operations in the same order, so a batch element must have the bits that it has in a
small batch, which the ring kernel takes; cut, its segments are others than the ring kernel's,
and sampled rows are held to the fp64 oracle (2e-3 on y, 1e-4 on states).
"""
import numpy as np
import pytest
import torch

from gpu_util import announce, check_against_oracle, has_gpu, to_device
from paper_2401_13660_amd.inputs import make_inputs
from plan_util import plan
from test_gpu_positions import check_states

pytestmark = [pytest.mark.gpu, pytest.mark.skipif(not has_gpu(), reason="needs a GPU")]


# an odd number of 16-timestep slices and an even one; dead lanes; 128 timesteps and more for each of 7 positions
@pytest.mark.parametrize("dtype,entry,L", [("f32", "fwd", 368), ("f32", "fwd", 512), ("f32", "states", 912), ("f32", "states", 1024),
                                           ("f32", "ckpt", 368), ("f32", "ckpt", 512), ("bf16", "ckpt", 368), ("bf16", "ckpt", 512)])
def test_same_bits_as_the_ring_kernel(dtype, entry, L):
    import paper_2401_13660_amd as mb
    dim, n = 2045, 32                                    # 256 chains each: 8,192
    gated, out_dtype = (True, torch.float32) if L in (368, 912) else (False, torch.bfloat16)
    kw = dict(dtype=dtype, gate=gated, out_bytes=2 if out_dtype == torch.bfloat16 else 4, ckpt=entry == "ckpt",
              npos=7 if entry == "states" else 0, h0=True)
    assert plan((1, dim, L), **kw).kernel == "ring" and plan((n, dim, L), **kw).kernel == "chunk"
    inp = make_inputs(1, dim, L, 16, dtype=dtype, seed=L, gated=gated, with_h0=True)
    t = to_device(inp)
    announce(f"chunk kernel, {dtype} {entry} ({n}, {dim}, {L}) gated={gated} out={out_dtype}")
    pos = torch.tensor([[-1], [0], [31], [L - 1], [L], [17], [L - 16]], dtype=torch.int32, device="cuda:0")

    def run(n):
        many = lambda x: None if x is None else x.expand(n, *x.shape[1:]).contiguous()
        h = many(t["h0"]).clone()                        # written over in place
        opt = dict(D=t["Dskip"], dt_bias=t["dt_bias"], z=many(t.get("z")), h0=h, h_last=h, out_dtype=out_dtype)
        if entry == "states":
            opt["positions"] = pos.expand(-1, n).contiguous()
        if entry == "ckpt":
            opt["return_ckpt"] = True
        return mb.scan_fwd(many(t["u"]), many(t["delta"]), t["A"], many(t["B"]), many(t["C"]), **opt)

    one, all_ = run(1), run(n)
    torch.cuda.synchronize()
    assert len(one) == len(all_)
    for i, (x, y) in enumerate(zip(one, all_)):
        x, y = torch.nan_to_num(x, nan=7.0), torch.nan_to_num(y, nan=7.0)
        if i == 2:                                       # (positions or slices, batch, dim, 16)
            x, y = x.transpose(0, 1), y.transpose(0, 1)
        assert torch.equal(y, x.expand_as(y)), i


# 160 chains in 26 segments of 2 pre-pass pieces, the last one of 16 timesteps more than an odd
# number of chunks, dead lanes; just over one chain per compute unit
@pytest.mark.parametrize("shape", [(1, 1277, 17 * 1024 + 16), (1, 2112, 8192)])
@pytest.mark.parametrize("entry", ["fwd", "states", "ckpt"])
def test_segments(shape, entry):
    import paper_2401_13660_amd as mb
    nb, dim, L = shape
    p = plan(shape, dtype="f32", ckpt=entry == "ckpt", npos=7 if entry == "states" else 0, h0=True)
    assert p.kernel == "chunk" and p.nseg > 8, p
    inp = make_inputs(nb, dim, L, 16, dtype="f32", seed=5, with_h0=True)
    rows = np.unique(np.concatenate([np.arange(0, dim, dim // 40), [dim - 1]]))
    t = to_device(inp)
    announce(f"chunk kernel, {p.nseg} segments, {entry} {shape}")
    state = t["h0"].clone()
    kw = dict(D=t["Dskip"], dt_bias=t["dt_bias"], z=t["z"], h0=state, h_last=state)
    pos = np.array([[-1], [0], [p.seg_len - 1], [p.seg_len], [3 * p.seg_len + 37], [L - 1], [L]], dtype=np.int32)
    if entry == "states":
        kw["positions"] = torch.from_numpy(pos).to("cuda:0")
    if entry == "ckpt":
        kw["return_ckpt"] = True
    res = mb.scan_fwd(t["u"], t["delta"], t["A"], t["B"], t["C"], **kw)
    torch.cuda.synchronize()
    check_against_oracle(inp, res[0], state, rows=rows)
    if entry == "states":
        check_states(inp, pos, res[2], state, rows=rows)
    if entry == "ckpt":
        at = (np.arange(L // 16) * 16 - 1)[::97, None].astype(np.int32)
        check_states(inp, at, res[2][::97].contiguous(), state, rows=rows)
