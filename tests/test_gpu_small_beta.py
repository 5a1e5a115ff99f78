"""d = 16 and 32: write gates down to 0 and to the smallest float32 numbers. A gate that small adds nothing to a state, so the
results are those of the oracle with it, at every token; the norm ||H_t||_F must not divide by it."""
import numpy as np
import pytest

import oracle
from paper_2511_21016_amd import binding, synth
from gka_testutil import pair_rel_err, to_device, to_host, upload_inputs

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("B,H,T", [(2, 3, 40), (2, 3, 330)])
@pytest.mark.parametrize("tiny", [1e-30, 1.2e-38, 8e-39, 1e-40, 1.5e-45, 0.0])
@pytest.mark.parametrize("d", [16, 32])
def test_tiny_write_gates(d, tiny, B, H, T):
    import torch
    w = synth.CFG2.scaled(d=d, B=B, H=H, T=T, n_iter=5, seed=77 + T)
    x = synth.make_inputs(w)
    beta = synth.make_gates(w)["beta"]
    for t in (5, 20, T - 3):
        beta[:, t, :] = tiny
    dev = upload_inputs(x, "bf16")
    print("tiny write gates", d, tiny, T, flush=True)
    o, ex = binding.gka_forward(dev["q"], dev["k"], dev["v"], dev["gate"], dev["lam"], w.n_iter, beta=to_device(beta, "f32"),
                                return_fro=True)
    torch.cuda.synchronize()
    ref, rex = oracle.forward(x["q"], x["k"], x["v"], x["gate"], x["lam"], w.n_iter, beta=beta, return_fro=True)
    assert pair_rel_err(to_host(o), ref) <= 2e-2                                # the stated bf16 tolerance
    assert np.abs(to_host(ex["fro"]) - rex["fro"]).max() <= 5e-3 * rex["fro"].max()


@pytest.mark.parametrize("tiny", [1e-8, 1e-18, 1e-20, 1e-22])
@pytest.mark.parametrize("d", [16, 32])
def test_tiny_states_under_the_rule(d, tiny):
    """A sequence whose first tokens are written with tiny gates only: ||H_t||_F^2 is a denormal number there, lambda_t and the
    solve's scale follow it, and the readout is of ordinary size."""
    import torch
    w = synth.CFG2.scaled(d=d, B=2, H=3, T=40, n_iter=5, seed=78)
    x = synth.make_inputs(w)
    beta = synth.make_gates(w)["beta"]
    beta[:, :2, :] = tiny
    dev = upload_inputs(x, "bf16")
    print("tiny states", d, tiny, flush=True)
    o, ex = binding.gka_forward(dev["q"], dev["k"], dev["v"], dev["gate"], None, w.n_iter, beta=to_device(beta, "f32"),
                                lambda_scale=0.05, return_fro=True)
    torch.cuda.synchronize()
    ref, rex = oracle.forward(x["q"], x["k"], x["v"], x["gate"], None, w.n_iter, beta=beta, lambda_scale=0.05, return_fro=True)
    fro, want = to_host(ex["fro"]), rex["fro"]
    # (a denormal square has 2^-149 / fro^2 of relative rounding: 1.4e-5 at 1e-20, 14 % at 1e-22)
    assert np.abs(fro / want - 1.0).max() <= 5e-3 + 1.5e-45 / tiny ** 2
    if tiny >= 1e-20:
        assert pair_rel_err(to_host(o), ref) <= 2e-2
    assert np.isfinite(to_host(o)).all()
