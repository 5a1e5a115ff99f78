"""GPU parity of the backward pass's reverse recurrences without an alpha-connection, where one walk serves both of them
(the tests with alpha in test_gpu_backward.py run them one after the other): edges of the 16-token tiles and of the
chunk, several segments of the walk, a write gate, a gate of 0 inside a chunk; against the backward oracle."""
import numpy as np
import pytest

from oracle import gka_backward_oracle as bwd
from paper_2511_21016_amd import binding, synth
from gka_testutil import to_device, to_host, upload_inputs

pytestmark = pytest.mark.gpu

# The stated bf16 tolerance of the backward pass. With float32 products in the two solves only the rounding of the
# stored operands is left: 2^-9 per operand of a few products (dk is a difference of sums several times its size).
TOL = {"bf16": 2e-2, "f32": 6e-3}


@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("T,compute", [(2, "f32"), (16, "bf16"), (17, "f32"), (63, "bf16"), (65, "f32"), (129, "bf16"),
                                       (321, "f32"), (1030, "bf16")])
def test_reverse_walk(T, compute, d):
    import torch
    w = synth.CFG2.scaled(B=2, H=3, T=T, d=d, n_iter=6, gate_mean=4.0, seed=9100 + T + d)
    x = synth.make_inputs(w)
    if T > 100:
        x["gate"][0, 77, 1] = 0.0                    # a packed sequence starts inside a chunk
    rng = np.random.default_rng(w.seed)
    dy = synth.round_to_bf16(rng.standard_normal(x["v"].shape).astype(np.float32))
    beta = synth.make_gates(w)["beta"] if T % 2 else None
    dev = upload_inputs(x, w.dtype)
    print("reverse", T, compute, d, flush=True)
    out = binding.gka_backward(dev["q"], dev["k"], dev["v"], dev["gate"], dev["lam"], to_device(dy, "bf16"), w.n_iter,
                               compute=binding.GKA_COMPUTE_F32 if compute == "f32" else binding.GKA_COMPUTE_BF16,
                               beta=None if beta is None else to_device(beta, "f32"))
    torch.cuda.synchronize()
    ref = bwd.backward(x["q"], x["k"], x["v"], x["gate"], x["lam"], dy, w.n_iter, beta=beta)
    errs = {}
    for name in ("dq", "dk", "dv", "dgate", "dlam") + (("dbeta",) if beta is not None else ()):
        got, want = to_host(out[name]), ref[name].copy()
        if name == "dgate":                          # (reported as 0 at a gate of 0)
            want[x["gate"] == 0.0] = 0.0
        axes = (1, 3) if got.ndim == 4 else (1,)
        errs[name] = float((np.abs(got - want).max(axis=axes) / np.abs(want).max(axis=axes)).max())
    print(errs)
    assert max(errs.values()) <= TOL[compute], errs
