"""GPU parity of the backward pass where its reverse scans over a pair's tokens are cut over several waves: blocks of 64
tokens, up to 16 waves, sequences of one block up to several blocks per wave, gates of 0 inside and at the edges of a wave's
range; against the fp64 oracle, with the layer's rule for lambda (whose own scan is cut alike) and without."""
import numpy as np
import pytest

from oracle import gka_backward_oracle as bwd
from paper_2511_21016_amd import binding, synth
from gka_testutil import to_device, to_host, upload_inputs

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("rule", [False, True])
@pytest.mark.parametrize("T", [2, 64, 65, 1024, 1025, 2113])
def test_backward_scans(T, rule):
    import torch
    w = synth.CFG2.scaled(d=64, B=1, H=2, T=T, n_iter=6, seed=3300 + T)
    x = synth.make_inputs(w)
    gate = x["gate"].copy()
    for t in (63, 64, 700, T - 128, T - 129, T - 64):
        if 0 < t < T and not rule:                   # (with the rule sequences of a few tokens are ill-conditioned)
            gate[:, t, 0] = 0.0
    dy = synth.round_to_bf16(np.random.default_rng(T).standard_normal(x["v"].shape).astype(np.float32))
    dev = upload_inputs(x, "bf16")
    print("backward_scans", T, rule, flush=True)
    out = binding.gka_backward(dev["q"], dev["k"], dev["v"], to_device(gate, "f32"), None if rule else dev["lam"],
                               to_device(dy, "bf16"), w.n_iter, compute=binding.GKA_COMPUTE_F32,
                               lambda_scale=0.05 if rule else 0.0)
    torch.cuda.synchronize()
    ref = bwd.backward(x["q"], x["k"], x["v"], gate, None if rule else x["lam"], dy, w.n_iter,
                       lambda_scale=0.05 if rule else 0.0)
    # The gate gradient's scan over several waves against the same scan by one wave (which a gate gradient that replaces the
    # gates takes): the terms are the same, only the float32 sums over up to T of them are ordered otherwise, which moves
    # a sum by at most T 2^-24 of its terms' magnitudes. The terms cancel: their rounding to bf16 moves the gradient by up to
    # 4e-2 against the oracle (below), so their magnitudes are up to 4e-2 / 2^-9 = 20 times the gradient.
    B, _, H, d = x["v"].shape
    gate_dev, dy_dev, spare = to_device(gate, "f32"), to_device(dy, "bf16"), [torch.empty_like(out[n]) for n in ("dq", "dk", "dv")]
    params = binding.make_params(B, H, T, d, w.n_iter, binding.GKA_BF16, binding.GKA_COMPUTE_F32,
                                 lambda_scale=0.05 if rule else 0.0)
    ws = torch.empty(max(binding.backward_workspace_bytes(params), 256), dtype=torch.uint8, device="cuda")
    status = binding.backward_raw(params, *(dev[n].data_ptr() for n in "qkv"), gate_dev.data_ptr(),
                                  None if rule else dev["lam"].data_ptr(), dy_dev.data_ptr(),
                                  *(g.data_ptr() for g in spare), gate_dev.data_ptr(), workspace=ws.data_ptr(),
                                  workspace_bytes=ws.numel())
    torch.cuda.synchronize()
    assert status == 0
    one, many = to_host(gate_dev), to_host(out["dgate"])
    diff = float((np.abs(many - one).max(axis=1) / np.abs(one).max(axis=1)).max())
    print("one wave against several:", diff, flush=True)
    assert diff <= 20 * max(T, 64) * 2.0 ** -24, diff
    # Against the oracle: the gate gradient and, with the rule, dk, at the tolerance stated for bf16 tensors. (The gate
    # gradient is a sum over up to T differences of terms rounded at 2^-9, which adds up as sqrt(T) of them.) With the rule
    # the sum takes in H_t k_t stored in bf16: 1.8e-2 at 1025 tokens, 4.4e-2 at 2113, summed by one wave as well: 6e-2
    # there.
    for name in ("dgate", "dk") if rule else ("dgate",):
        got, want = to_host(out[name]), ref[name].copy()
        if name == "dgate":                          # (reported as 0 at a gate of 0)
            want[gate == 0.0] = 0.0
        axes = (1, 3) if got.ndim == 4 else (1,)
        err = float((np.abs(got - want).max(axis=axes) / np.abs(want).max(axis=axes)).max())
        assert err <= (6e-2 if rule and name == "dgate" and T > 2000 else 2e-2), (name, err)
