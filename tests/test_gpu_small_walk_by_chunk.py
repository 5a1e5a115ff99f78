"""GPU parity of the walk of the head dimensions 16 and 32 whose four waves take the four tiles of a chunk (where chunks are few)
against the fp64 oracle: last chunks of one token, of part of a tile, of one to four tiles; initial states and the layer's
variants; gates of 0 inside a chunk. Its choice against the other walks, on the CPU."""
import numpy as np
import pytest

import oracle
from paper_2511_21016_amd import binding, synth
from gka_testutil import pair_rel_err, to_device, to_host, upload_inputs
from hip_recorder import record

CHUNKS = [(16, 25, 5, 209), (16, 60, 1, 257), (16, 10, 6, 271), (16, 10, 5, 288), (16, 1, 3, 1000), (16, 20, 10, 305),
          (32, 2, 3, 161), (32, 1, 4, 193), (32, 2, 2, 207), (32, 1, 1, 256), (32, 1, 3, 1000), (32, 30, 8, 497)]


@pytest.mark.parametrize("d,B,H,T,by_chunk", [(*s, True) for s in CHUNKS] + [
    (16, 1, 1, 256, False), (16, 2, 2, 305, False), (16, 8, 15, 197, True), (16, 16, 16, 150, False), (32, 1, 1, 160, False), (16, 60, 10, 400, False),
    (32, 64, 10, 257, False), (16, 4, 4, 128, False)])
def test_kernel_choice(d, B, H, T, by_chunk):
    calls = record(f"""
X = 1 << 40
p = binding.make_params({B}, {H}, {T}, {d}, 5, binding.GKA_BF16, binding.GKA_COMPUTE_BF16)
st = binding.forward_raw(p, X, X + 1, X + 2, X, X, X + 3, workspace=X, workspace_bytes=1 << 50)
assert st == binding.GKA_OK, binding.status_string(st)
""")
    assert calls[-1]["kernel"] == "small_walk_kernel"
    assert by_chunk == calls[-1]["mangled"].split("EEE")[0].endswith("Li2")       # WALK_CHUNK


@pytest.mark.gpu
@pytest.mark.parametrize("variants", [False, True])
@pytest.mark.parametrize("d,B,H,T", CHUNKS)
def test_walk_by_chunk(d, B, H, T, variants):
    import torch
    w = synth.CFG2.scaled(d=d, B=B, H=H, T=T, n_iter=5, seed=6700 + d + T)
    x = synth.make_inputs(w)
    x["gate"][0, 70, 0] = x["gate"][0, T - 2, 0] = 0.0
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
        x["gate"][0, 70, 0] = x["gate"][0, T - 2, 0] = 0.3      # (the rule alone is ill-conditioned for a single token)
        dev["gate"] = to_device(x["gate"], "f32")
    lam = (None, None) if variants else (x["lam"], dev["lam"])
    print("walk by chunk", d, B, H, T, variants, flush=True)
    o, ex = binding.gka_forward(dev["q"], dev["k"], dev["v"], dev["gate"], lam[1], w.n_iter, return_fro=True,
                                return_state=True, return_xhat=True, **dkw)
    torch.cuda.synchronize()
    ref, rex = oracle.forward(x["q"], x["k"], x["v"], x["gate"], lam[0], w.n_iter, return_fro=True, return_state=True,
                              return_xhat=True, **kw)
    # worst pair: the stated bf16 tolerance. 2-norm: rounding is uniform within 2^-9 of a value, 1.1e-3; the output once, the
    # update of every pass and the masked products, which the solve adds up: twice the output's share on top
    assert pair_rel_err(to_host(o), ref) <= 2e-2
    assert np.linalg.norm(to_host(o) - ref) <= 6e-3 * np.linalg.norm(ref)
    assert np.abs(to_host(ex["fro"]) - rex["fro"]).max() <= 5e-3 * rex["fro"].max()
    assert pair_rel_err(to_host(ex["xhat"]), rex["xhat"]) <= 2e-2
    # weighted rows as bf16 value + remainder: 2^-17 of a term
    for n in ("H_final", "U_final"):
        assert np.abs(to_host(ex[n]) - rex[n]).max() <= 1e-4 * np.abs(rex[n]).max(), n
