"""A seeded sweep of random configurations through the forward and the backward,
each compared with the fp64 oracle at the bars of tests/parity.py (forward) and
tests/test_gpu_bwd.py (backward).

The cases are drawn once from a fixed seed, so the list and each case's inputs
are the same on every run.  They cover:
- batch 1-4 and dim 1-300 (dead lanes in the last 8-channel group whenever
  dim % 8 != 0);
- forward lengths 0-2100, multiples of 16 and others; dstate 16, and 1, 2, 4 or 8 on the
  row-per-thread kernel;
- forward lengths 2048-6000 of few rows, which are cut into time segments;
- backward lengths that are multiples of 16 up to 1600, dstate 16;
- fp32 or bf16 activations, fp32 or bf16 outputs;
- each optional input (z, h0, Dskip, dt_bias, dh_last) present or absent;
- A of the S4D kind or random; softplus on, or off with a small positive delta
  and dt_bias.
"""
import numpy as np
import pytest
import torch

from gpu_util import announce, check_against_oracle, gpu_fwd, has_gpu
from parity import TOL_Y, TOL_Y_BF16_OUT
from plan_util import plan
from paper_2401_13660_amd.inputs import bf16_bits_to_f32, f32_to_bf16_bits, make_inputs

pytestmark = [pytest.mark.gpu, pytest.mark.skipif(not has_gpu(), reason="needs a GPU")]


def _draw(rng, backward: bool) -> dict:
    c = dict(batch=int(rng.integers(1, 5)), dim=int(rng.integers(1, 301)),
             dtype=str(rng.choice(["f32", "bf16"])), gated=bool(rng.random() < 0.7),
             with_h0=bool(rng.random() < 0.5), with_D=bool(rng.random() < 0.8),
             with_bias=bool(rng.random() < 0.8), A_kind=str(rng.choice(["s4d", "random"])),
             softplus=bool(rng.random() < 0.8), out_bf16=bool(rng.random() < 0.3))
    if backward:
        c.update(L=16 * int(rng.integers(1, 101)), N=16, with_dhl=bool(rng.random() < 0.6))
    else:
        tiled = rng.random() < 0.6
        c["L"] = 16 * int(rng.integers(0, 132)) if tiled else int(rng.integers(0, 2101))
        c["N"] = 16 if tiled else int(rng.choice([1, 2, 4, 8, 16]))
    return c


def _cases(seed: int, n: int, backward: bool):
    rng = np.random.default_rng(seed)
    return [_draw(rng, backward) for _ in range(n)]


def _case_id(c: dict) -> str:
    opts = "".join(k for k, on in (("z", c["gated"]), ("h", c["with_h0"]), ("D", c["with_D"]),
                                    ("b", c["with_bias"]), ("s", c["softplus"]), ("o", c["out_bf16"])) if on)
    return f"{c['batch']}x{c['dim']}x{c['L']}-N{c['N']}-{c['dtype']}-{c['A_kind']}-{opts}"


def _inputs(c: dict, seed: int):
    inp = make_inputs(c["batch"], c["dim"], c["L"], c["N"], dtype=c["dtype"], seed=seed, gated=c["gated"],
                      with_h0=c["with_h0"], with_D=c["with_D"], with_bias=c["with_bias"], A_kind=c["A_kind"])
    if not c["softplus"]:
        # dlt = delta + dt_bias as given: keep both small and positive (a negative
        # dlt makes abar = exp(dlt A) > 1 and the state overflow fp32)
        if inp.dt_bias is not None:
            inp.dt_bias = (np.abs(inp.dt_bias) * np.float32(0.01)).astype(np.float32)
        if c["dtype"] == "bf16":
            d = np.abs(bf16_bits_to_f32(inp.delta)).astype(np.float32) * np.float32(0.05)
            inp.delta = f32_to_bf16_bits(d).reshape(inp.delta.shape)
        else:
            inp.delta = (np.abs(inp.delta) * np.float32(0.05)).astype(np.float32)
    return inp


def _segment_cases(seed: int, n: int):
    rng = np.random.default_rng(seed)
    cases = [_draw(rng, False) for _ in range(n)]
    for c in cases:
        c.update(N=16, batch=int(rng.integers(1, 3)), dim=int(rng.integers(1, 200)), L=int(rng.integers(2048, 6001)))
        if rng.random() < 0.4:
            c["L"] -= c["L"] % 16
    return cases


FWD_CASES = _cases(2401, 32, backward=False)
SEG_CASES = _segment_cases(1366, 10)
BWD_CASES = _cases(13660, 16, backward=True)


@pytest.mark.parametrize("i", range(len(FWD_CASES)), ids=[_case_id(c) for c in FWD_CASES])
def test_random_forward(i):
    c = FWD_CASES[i]
    inp = _inputs(c, seed=100 + i)
    announce(f"random forward {i}: {_case_id(c)}")
    out = torch.bfloat16 if c["out_bf16"] else torch.float32
    y, h = gpu_fwd(inp, out_dtype=out, delta_softplus=c["softplus"])
    check_against_oracle(inp, y, h, tol_y=TOL_Y_BF16_OUT if c["out_bf16"] else TOL_Y,
                         delta_softplus=c["softplus"])


@pytest.mark.parametrize("i", range(len(SEG_CASES)), ids=[_case_id(c) for c in SEG_CASES])
def test_random_segmented_forward(i):
    c = SEG_CASES[i]
    assert plan((c["batch"], c["dim"], c["L"]), aligned=c["L"] % 16 == 0).nseg > 1
    inp = _inputs(c, seed=400 + i)
    announce(f"random segmented forward {i}: {_case_id(c)}")
    out = torch.bfloat16 if c["out_bf16"] else torch.float32
    y, h = gpu_fwd(inp, out_dtype=out, delta_softplus=c["softplus"])
    check_against_oracle(inp, y, h, tol_y=TOL_Y_BF16_OUT if c["out_bf16"] else TOL_Y,
                         delta_softplus=c["softplus"])


@pytest.mark.parametrize("i", range(len(BWD_CASES)), ids=[_case_id(c) for c in BWD_CASES])
def test_random_backward(i):
    from test_gpu_bwd import grads_case
    c = BWD_CASES[i]
    inp = _inputs(c, seed=200 + i)
    announce(f"random backward {i}: {_case_id(c)} dh_last={c['with_dhl']}")
    grads_case(inp, with_dhl=c["with_dhl"], out_dtype=torch.bfloat16 if c["out_bf16"] else torch.float32,
               delta_softplus=c["softplus"], seed=300 + i)
