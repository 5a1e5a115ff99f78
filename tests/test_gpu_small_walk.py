"""GPU parity of the walk kernel of the head dimensions 16 and 32 (bf16 tensors and operands) against the fp64 oracle, at
the edges of its tiles (16 tokens) and on problems of every way in which its walks are cut: a wave per tile from the
sequence's start, a workgroup of four waves per chunk, one wave per chunk, one walk per pair."""
import numpy as np
import pytest

import oracle
from paper_2511_21016_amd import binding, synth
from gka_testutil import to_device, to_host, upload_inputs

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("variants", [False, True])
@pytest.mark.parametrize("d,B,H,T", [
    (16, 2, 3, 1), (16, 2, 2, 17), (16, 1, 3, 64), (32, 2, 3, 15), (32, 1, 2, 128), (32, 2, 3, 250),     # tile by tile
    (16, 2, 3, 321), (16, 32, 5, 257), (32, 1, 3, 257),              # four waves per chunk
    (16, 15, 12, 390), (32, 10, 15, 401), (16, 16, 12, 705),
    (32, 19, 10, 721), (16, 60, 10, 401), (32, 64, 10, 257),         # one wave per chunk
    (16, 41, 25, 65), (16, 128, 16, 145), (32, 64, 16, 129)])        # one walk per pair
def test_small_walk(d, B, H, T, variants):
    import torch
    w = synth.CFG2.scaled(d=d, B=B, H=H, T=T, n_iter=5, seed=6100 + d + T)
    x = synth.make_inputs(w)
    dev = upload_inputs(x, "bf16")
    kw, dkw = {}, {}
    if variants:
        g = synth.make_gates(w)
        rng = np.random.default_rng(d + T)
        A = rng.standard_normal((B, H, d, 8)) / np.sqrt(d)
        kw = dict(beta=g["beta"], alpha=g["alpha"], lambda_scale=0.05,
                  H_init=(A @ np.transpose(A, (0, 1, 3, 2))).astype(np.float32),
                  U_init=(rng.standard_normal((B, H, d, d)) / d).astype(np.float32))
        dkw = {n: v if n == "lambda_scale" else to_device(v, "f32") for n, v in kw.items()}
    lam = (None, None) if variants else (x["lam"], dev["lam"])
    print("small_walk", d, B, H, T, variants, flush=True)
    o, ex = binding.gka_forward(dev["q"], dev["k"], dev["v"], dev["gate"], lam[1], w.n_iter, return_fro=True,
                                return_state=True, return_xhat=variants, **dkw)
    torch.cuda.synchronize()
    ref, rex = oracle.forward(x["q"], x["k"], x["v"], x["gate"], lam[0], w.n_iter, return_fro=True, return_state=True,
                              return_xhat=variants, **kw)
    # Rounding to bf16 is uniform within 2^-9 of a value, 1.1e-3 in the 2-norm: the output once, the update delta of every
    # pass and the masked products, which the solve adds up and amplifies on some tokens (two times the output's share in
    # all). A token gone wrong in one pair does not show in that norm of all of them: it does in the pair's own, as T^-1/2,
    # 3.7e-2 at the longest here. (The largest difference of the worst of thousands of pairs would not do: it is that of the
    # one token whose solve amplifies rounding most, 2.4e-2 of the pair's largest value here.)
    diff = to_host(o) - ref
    pair = np.sqrt((diff ** 2).sum(axis=(1, 3)) / (ref ** 2).sum(axis=(1, 3)))
    assert pair.max() <= 2e-2, pair.max()
    assert np.linalg.norm(to_host(o) - ref) <= 6e-3 * np.linalg.norm(ref)
    assert np.abs(to_host(ex["fro"]) - rex["fro"]).max() <= 5e-3 * rex["fro"].max()
    if variants:
        assert np.abs(to_host(ex["xhat"]) - rex["xhat"]).max() <= 2e-2 * np.abs(rex["xhat"]).max()
    for n in ("H_final", "U_final"):
        assert np.abs(to_host(ex[n]) - rex[n]).max() <= 5e-3 * np.abs(rex[n]).max(), n
