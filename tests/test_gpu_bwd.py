"""GPU parity of mb_scan_bwd against the fp64 oracle's backward.

Every gradient is compared on the same input bits under the metric of
tests/parity.py.  Bars (fp32 arithmetic and fp32 gradients, against the fp64
oracle): 1e-4 for the per-element gradients du, ddelta, dz, for dB and dC
(sums over channels) and for dh0; 2e-4 for dA, dDskip and dbias, which sum
over every (batch, time) of a channel (up to 32,768 terms at the 972M layer
shape, where 2e-5 is observed).  A bf16 gradient output adds one bf16
rounding (2^-8).
"""
import numpy as np
import pytest
import torch

import oracle
from gpu_util import announce, dev_tensor, has_gpu
from parity import rel_err
from plan_util import plan
from paper_2401_13660_amd.inputs import make_inputs, workload

pytestmark = [pytest.mark.gpu, pytest.mark.skipif(not has_gpu(), reason="needs a GPU")]

TOL = dict(du=1e-4, ddelta=1e-4, dz=1e-4, dB=1e-4, dC=1e-4, dA=2e-4, dD=2e-4, ddt_bias=2e-4, dh0=1e-4)
ORACLE_NAME = dict(du="du", ddelta="ddelta", dz="dz", dA="dA", dB="dB", dC="dC", dD="dD", ddt_bias="dbias",
                   dh0="dh0")


def grads_case(inp, *, with_dhl=True, out_dtype=torch.float32, delta_softplus=True, seed=60, rows=None):
    import paper_2401_13660_amd as mb
    t = {k: dev_tensor(v) for k, v in inp.arrays().items()}
    rng = np.random.default_rng(seed)
    dy = rng.standard_normal(inp.u.shape).astype(np.float32)
    if out_dtype == torch.bfloat16:
        from paper_2401_13660_amd.inputs import bf16_bits_to_f32, f32_to_bf16_bits
        dy_bits = f32_to_bf16_bits(dy).reshape(dy.shape)
        dy = bf16_bits_to_f32(dy_bits).reshape(dy.shape)
        dy_dev = dev_tensor(dy_bits)
    else:
        dy_dev = dev_tensor(dy)
    dhl = rng.standard_normal((inp.batch, inp.dim, inp.dstate)).astype(np.float32) if with_dhl else None
    g = mb.scan_bwd(t["u"], t["delta"], t["A"], t["B"], t["C"], dy_dev, D=t.get("Dskip"),
                    dt_bias=t.get("dt_bias"), z=t.get("z"), h0=t.get("h0"), dh_last=dev_tensor(dhl),
                    delta_softplus=delta_softplus)
    torch.cuda.synchronize()
    ref = oracle.default().scan_bwd(inp.u, inp.delta, inp.A, inp.B, inp.C, dy, z=inp.z, Dskip=inp.Dskip,
                                    dt_bias=inp.dt_bias, h0=inp.h0, dh_last=dhl, delta_softplus=delta_softplus,
                                    dtype=inp.dtype)
    errs = {}
    bf = out_dtype == torch.bfloat16
    for k, gv in g.items():
        r = ref[ORACLE_NAME[k]]
        if gv is None or r is None:
            assert (gv is None) == (r is None or k == "dh0"), k
            continue
        gv = gv.float().cpu().numpy().astype(np.float64)
        if rows is not None and k in ("du", "ddelta", "dz", "dh0"):
            gv = gv.reshape(inp.batch * inp.dim, -1)[rows]
            r = r.reshape(inp.batch * inp.dim, -1)[rows]
        errs[k] = rel_err(gv, r)
    print("[bwd errors]", {k: f"{v:.2e}" for k, v in errs.items()}, flush=True)
    for k, e in errs.items():
        tol = TOL[k] + (2.0 ** -8 if bf and k in ("du", "ddelta", "dz") else 0.0)
        assert e <= tol, f"{k}: relative error {e:.3e} > {tol:.1e}"
    return errs


# (batch, dim, L): one chunk; several chunks with dead lanes in the last
# 8-channel group; a long reverse carry; a single ragged group; one group; more
# than 1,024 channel groups (more waves than SIMDs), with and without dead lanes;
# at least 1,536 groups, a multiple of 4 per batch element, where the 4 waves of a
# workgroup also sum their dB/dC terms with each other, with and without dead lanes;
# few rows and a long sequence, cut into time segments (3 segments, the last one
# shorter, whose aggregate pre-pass runs in 4 pieces per segment, one of them past
# the end; with 5 rows the aggregate planes are only 8-byte aligned; 8 segments
# whose waves also take the workgroup sum).
@pytest.mark.parametrize("shape", [(2, 196, 16), (3, 101, 48), (2, 197, 1008), (1, 5, 1008), (1, 5, 32), (1, 8, 16),
                                   (9, 1001, 32), (9, 1024, 16), (12, 1024, 16), (12, 1020, 32),
                                   (2, 1024, 2048)])
@pytest.mark.parametrize("dtype", ["bf16", "f32"])
def test_bwd_shapes(shape, dtype):
    inp = make_inputs(*shape, 16, dtype=dtype, seed=61, with_h0=True)
    announce(f"bwd {shape} {dtype}")
    grads_case(inp)


@pytest.mark.parametrize("gated,with_h0,with_dhl", [(False, False, False), (True, False, True),
                                                    (False, True, False)])
def test_bwd_options(gated, with_h0, with_dhl):
    inp = make_inputs(2, 64, 256, 16, dtype="bf16", seed=62, gated=gated, with_h0=with_h0)
    announce(f"bwd gated={gated} h0={with_h0} dh_last={with_dhl}")
    grads_case(inp, with_dhl=with_dhl)


def test_bwd_no_skip_no_bias_no_softplus():
    from paper_2401_13660_amd.inputs import bf16_bits_to_f32, f32_to_bf16_bits
    inp = make_inputs(2, 64, 256, 16, dtype="bf16", seed=63, with_D=False, with_bias=False)
    # without softplus Delta = delta_raw is used as given: keep it positive
    vals = np.abs(bf16_bits_to_f32(inp.delta).reshape(inp.u.shape)) * 0.1 + 0.01
    inp.delta = f32_to_bf16_bits(vals.astype(np.float32)).reshape(inp.u.shape)
    announce("bwd no skip, no bias, no softplus")
    grads_case(inp, delta_softplus=False)


def test_bwd_random_A_and_bf16_gradients():
    inp = make_inputs(2, 96, 512, 16, dtype="bf16", seed=64, with_h0=True, A_kind="random")
    announce("bwd random A, bf16 dy and gradients")
    grads_case(inp, out_dtype=torch.bfloat16)


def test_bwd_empty_sequence():
    """L = 0: the state passes straight through (dh0 = dh_last) and every parameter
    gradient is zero; a batch of 0 rows is a no-op."""
    import paper_2401_13660_amd as mb
    dev = "cuda:0"
    nb, dim, N = 2, 24, 16
    z3 = lambda *sh, dt=torch.bfloat16: torch.zeros(sh, dtype=dt, device=dev)
    A = -torch.arange(1, N + 1, dtype=torch.float32, device=dev).repeat(dim, 1)
    dhl = torch.randn((nb, dim, N), generator=torch.Generator().manual_seed(5)).to(dev)
    announce("bwd L = 0")
    g = mb.scan_bwd(z3(nb, dim, 0), z3(nb, dim, 0), A, z3(nb, N, 0), z3(nb, N, 0),
                    z3(nb, dim, 0, dt=torch.float32), D=torch.ones(dim, device=dev),
                    dt_bias=torch.zeros(dim, device=dev), dh_last=dhl)
    torch.cuda.synchronize()
    assert torch.equal(g["dh0"], dhl)
    for k in ("dA", "dD", "ddt_bias"):
        assert torch.count_nonzero(g[k]) == 0, k
    g0 = mb.scan_bwd(z3(0, dim, 32), z3(0, dim, 32), A, z3(0, N, 32), z3(0, N, 32),
                     z3(0, dim, 32, dt=torch.float32))
    torch.cuda.synchronize()
    assert g0["du"].numel() == 0
    assert torch.count_nonzero(g0["dA"]) == 0, "dA over an empty batch must be zero"


@pytest.mark.parametrize("shape", [(2, 128, 512), (9, 1001, 64), (12, 1020, 64), (2, 1024, 2048)],
                         ids=["small_two_segments", "many_groups", "workgroup_sum", "segments_and_workgroup_sum"])
def test_bwd_deterministic(shape):
    import paper_2401_13660_amd as mb
    inp = make_inputs(*shape, 16, dtype="bf16", seed=65, with_h0=True)
    t = {k: dev_tensor(v) for k, v in inp.arrays().items()}
    dy = torch.randn(inp.u.shape, generator=torch.Generator().manual_seed(0)).to("cuda:0")
    announce("bwd determinism")
    outs = [mb.scan_bwd(t["u"], t["delta"], t["A"], t["B"], t["C"], dy, D=t["Dskip"], dt_bias=t["dt_bias"],
                        z=t["z"], h0=t["h0"]) for _ in range(2)]
    torch.cuda.synchronize()
    for k in outs[0]:
        if outs[0][k] is not None:
            assert torch.equal(outs[0][k], outs[1][k]), f"{k} differs between runs"


@pytest.mark.parametrize("name", ["mambabyte353m_L8192", "mambabyte972m_L8192"])
def test_bwd_layer_every_row(name):
    """The 353M and 972M layer shapes at full size: every gradient of every row."""
    inp = workload(name, seed=0)
    announce(f"bwd {name} {inp.u.shape}, every row")
    grads_case(inp, with_dhl=False)


# ---- the training pair: the forward stores the checkpoints, the backward reads them

def _fwd_ckpt(t):
    import paper_2401_13660_amd as mb
    kw = dict(D=t.get("Dskip"), dt_bias=t.get("dt_bias"), z=t.get("z"), h0=t.get("h0"), return_last_state=True)
    y, hl, ck = mb.scan_fwd(t["u"], t["delta"], t["A"], t["B"], t["C"], return_ckpt=True, **kw)
    y0, hl0 = mb.scan_fwd(t["u"], t["delta"], t["A"], t["B"], t["C"], **kw)
    torch.cuda.synchronize()
    assert torch.equal(y, y0), "storing checkpoints changed y"
    assert torch.equal(hl, hl0), "storing checkpoints changed h_last"
    return ck


# (batch, dim, L): dead lanes; an odd number of slices; few chains, uncut and cut into time
# segments (whose waves start from a folded state); the 353M layer's width, 1,024 chains.
@pytest.mark.parametrize("shape", [(2, 196, 512), (3, 100, 208), (1, 64, 1024), (1, 64, 4096), (4, 2048, 1024)])
@pytest.mark.parametrize("dtype", ["bf16", "f32"])
def test_fwd_checkpoints_match_oracle_states(shape, dtype):
    """ck[k] is the state before timestep 16k: the oracle's state at position 16k - 1."""
    nb, dim, L = shape
    assert (plan(shape, ckpt=True).nseg > 1) == (L == 4096)
    inp = make_inputs(nb, dim, L, 16, dtype=dtype, seed=67, with_h0=True)
    announce(f"forward checkpoints {shape} {dtype}")
    ck = _fwd_ckpt({k: dev_tensor(v) for k, v in inp.arrays().items()})
    pos = np.repeat((np.arange(L // 16) * 16 - 1)[:, None], nb, axis=1).astype(np.int32)
    _, _, h_ref = oracle.scan_inputs(inp, positions=pos)                  # (L/16, rows, N)
    got = ck.cpu().numpy().reshape(L // 16, nb * dim, 16).astype(np.float64)
    assert np.array_equal(got[0], inp.h0.reshape(nb * dim, 16).astype(np.float64)), "ck[0] is not h0"
    e = rel_err(got, h_ref)
    print(f"[ck error] {e:.2e}", flush=True)
    assert e <= 1e-4, f"checkpoints: relative error {e:.3e}"


@pytest.mark.parametrize("shape,gated", [((2, 196, 512), True), ((1, 64, 1024), False), ((1, 64, 4096), False), ((9, 1001, 64), True),
                                         ((12, 1024, 32), True), ((4, 2048, 256), True)])
def test_bwd_from_forward_checkpoints(shape, gated):
    """The backward from the forward's checkpoints: oracle parity, and the same
    gradients as the backward that recomputes its checkpoints."""
    import paper_2401_13660_amd as mb
    inp = make_inputs(*shape, 16, dtype="bf16", seed=68, with_h0=True, gated=gated)
    announce(f"bwd from forward checkpoints {shape} gated={gated}")
    t = {k: dev_tensor(v) for k, v in inp.arrays().items()}
    ck = _fwd_ckpt(t)
    dy = torch.randn(inp.u.shape, generator=torch.Generator().manual_seed(3)).to("cuda:0")
    kw = dict(D=t.get("Dskip"), dt_bias=t.get("dt_bias"), z=t.get("z"), h0=t.get("h0"))
    g_ck = mb.scan_bwd(t["u"], t["delta"], t["A"], t["B"], t["C"], dy, ck=ck, **kw)
    g_re = mb.scan_bwd(t["u"], t["delta"], t["A"], t["B"], t["C"], dy, **kw)
    torch.cuda.synchronize()
    same = all(torch.equal(g_ck[k], g_re[k]) for k in g_ck if g_ck[k] is not None)
    print(f"[bwd from ck] bit-identical to the recomputing call: {same}", flush=True)
    for k in g_ck:
        if g_ck[k] is None:
            continue
        e = rel_err(g_ck[k].double().cpu().numpy(), g_re[k].double().cpu().numpy())
        assert e <= 1e-5, f"{k}: {e:.3e} between the two checkpoint sources"
    ref = oracle.default().scan_bwd(inp.u, inp.delta, inp.A, inp.B, inp.C, dy.cpu().numpy(), z=inp.z,
                                    Dskip=inp.Dskip, dt_bias=inp.dt_bias, h0=inp.h0, dtype=inp.dtype)
    for k in g_ck:
        if g_ck[k] is None:
            continue
        e = rel_err(g_ck[k].double().cpu().numpy(), ref[ORACLE_NAME[k]])
        assert e <= TOL[k], f"{k}: relative error {e:.3e} > {TOL[k]:.1e}"
