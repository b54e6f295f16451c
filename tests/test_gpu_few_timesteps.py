"""A few timesteps of many rows: the row kernel takes them without a first state or positions, the ring
kernel with either.  Its sums are formed in the ring kernel's order, so that recording states
changes no bit, and sampled rows are held to the fp64 oracle."""
import dataclasses

import numpy as np
import pytest
import torch

from gpu_util import announce, check_against_oracle, has_gpu, to_device
from paper_2401_13660_amd.inputs import make_inputs
from plan_util import plan

pytestmark = [pytest.mark.gpu, pytest.mark.skipif(not has_gpu(), reason="needs a GPU")]


# dead lanes; the smallest and largest lengths of each type
@pytest.mark.parametrize("dtype,out_dtype,L", [("bf16", torch.float32, 1), ("bf16", torch.bfloat16, 2), ("bf16", torch.float32, 7),
                                               ("bf16", torch.bfloat16, 8), ("f32", torch.float32, 1), ("f32", torch.bfloat16, 2),
                                               ("f32", torch.float32, 3), ("f32", torch.float32, 4)])
@pytest.mark.parametrize("softplus", [True, False])
def test_row_kernel_has_the_ring_kernels_bits(dtype, out_dtype, L, softplus):
    import paper_2401_13660_amd as mb
    nb, dim = 192, 1621                                  # 203 chains each: 152 per compute unit
    kw = dict(dtype=dtype, out_bytes=2 if out_dtype == torch.bfloat16 else 4)
    assert plan((nb, dim, L), **kw).kernel == "row" and plan((nb, dim, L), npos=3, **kw).kernel == "ring"
    inp = make_inputs(nb, dim, L, 16, dtype=dtype, seed=L, with_bias=softplus)
    if not softplus:                                     # timesteps as they are: none negative
        inp = dataclasses.replace(inp, delta=inp.delta & 0x7FFF if dtype == "bf16" else np.abs(inp.delta))
    t = to_device(inp)
    announce(f"few timesteps, {dtype} ({nb}, {dim}, {L}) out={out_dtype} softplus={softplus}")
    args = (t["u"], t["delta"], t["A"], t["B"], t["C"])
    opt = dict(D=t["Dskip"], dt_bias=t.get("dt_bias"), z=t["z"], delta_softplus=softplus, out_dtype=out_dtype, return_last_state=True)
    y, h = mb.scan_fwd(*args, **opt)
    pos = torch.tensor([[L - 1], [-1], [0]], dtype=torch.int32, device="cuda:0").expand(-1, nb).contiguous()
    y_at, h_last, h_at = mb.scan_fwd(*args, positions=pos, **opt)
    torch.cuda.synchronize()
    assert torch.equal(y, y_at) and torch.equal(h, h_last)
    assert torch.equal(h_at[0], h) and not h_at[1].any()
    rows = np.unique(np.concatenate([np.arange(0, nb * dim, nb * dim // 50), [nb * dim - 1]]))
    check_against_oracle(inp, y, h, rows=rows, tol_y=2e-3 if out_dtype == torch.float32 else 2e-3 + 2 ** -8, delta_softplus=softplus)
