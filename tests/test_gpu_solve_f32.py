"""GPU parity of the per-chunk solve with float32 products (d = 64, 128 and, on GKA_PATH_AUTO, 256) against the fp64
oracle, at the edges of its token tiles (16 tokens) and on problems large enough for each of its workgroup sizes (16 and 32
tokens)."""
import numpy as np
import pytest

import oracle
from paper_2511_21016_amd import binding, synth
from gka_testutil import pair_rel_err, to_device, to_host, upload_inputs

pytestmark = pytest.mark.gpu

# Float32 sums of some hundred terms, amplified by a solve of condition number (L / mu) below 1e3: 1e-4 of the largest
# value (the bound of every float32 path of this library); bf16 outputs round at 2^-9 of a value on top of it.
TOL = {"f32": 1e-4, "bf16": 1e-4 + 2.0 ** -8}


@pytest.mark.parametrize("variants", [False, True])
@pytest.mark.parametrize("d,dtype,B,H,T", [
    (64, "f32", 2, 3, 1), (64, "f32", 2, 2, 79), (64, "f32", 7, 19, 97), (64, "f32", 9, 16, 191),
    (128, "f32", 1, 2, 16), (128, "f32", 1, 3, 145), (128, "bf16", 5, 30, 65), (128, "f32", 11, 13, 113),
    (256, "f32", 1, 2, 129), (256, "bf16", 2, 3, 193), (256, "f32", 1, 1, 321), (256, "f32", 6, 8, 177)])
def test_solve_f32(d, dtype, B, H, T, variants):
    base = synth.CFG2 if dtype == "bf16" else synth.CFG1
    w = base.scaled(d=d, B=B, H=H, T=T, n_iter=6, seed=7000 + d + T)
    x = synth.make_inputs(w)
    dev = upload_inputs(x, dtype)
    kw, dkw = {}, {}
    if variants:
        g = synth.make_gates(w)
        rng = np.random.default_rng(d + T)
        A = rng.standard_normal((B, H, d, 8)) / np.sqrt(d)
        init = {"H_init": (A @ np.transpose(A, (0, 1, 3, 2))).astype(np.float32),
                "U_init": (rng.standard_normal((B, H, d, d)) / d).astype(np.float32)}
        kw = dict(beta=g["beta"], alpha=g["alpha"], lambda_scale=0.05, **init)
        dkw = {n: v if n == "lambda_scale" else to_device(v, "f32") for n, v in kw.items()}
    lam = (None, None) if variants else (x["lam"], dev["lam"])
    print("solve_f32", d, dtype, B, H, T, variants, flush=True)
    import torch
    o, ex = binding.gka_forward(dev["q"], dev["k"], dev["v"], dev["gate"], lam[1], w.n_iter,
                                compute=binding.GKA_COMPUTE_F32, return_fro=True, return_state=True,
                                return_xhat=variants, **dkw)
    torch.cuda.synchronize()
    ref, rex = oracle.forward(x["q"], x["k"], x["v"], x["gate"], lam[0], w.n_iter, return_fro=True, return_state=True,
                              return_xhat=variants, **kw)
    assert pair_rel_err(to_host(o), ref) <= TOL[dtype]
    assert np.abs(to_host(ex["fro"]) - rex["fro"]).max() <= 1e-5 * rex["fro"].max()
    if variants:
        assert pair_rel_err(to_host(ex["xhat"]), rex["xhat"]) <= 1e-4
    for n in ("H_final", "U_final"):
        assert np.abs(to_host(ex[n]) - rex[n]).max() <= 1e-5 * np.abs(rex[n]).max(), n
