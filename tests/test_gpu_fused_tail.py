"""The fused forward kernel where the sequence ends inside a chunk, or with a chunk that has no second one beside it: no passes and no
readout for tokens that do not exist. A token's output does not depend on later ones: the same bits as in a longer sequence."""
import numpy as np
import pytest

from paper_2511_21016_amd import binding, synth
from gka_testutil import to_device, upload_inputs

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("T", [1, 15, 16, 17, 48, 63, 64, 65, 112, 127, 129, 144, 176, 192, 200])
@pytest.mark.parametrize("variants,split", [(False, False), (True, False), (False, True), (True, True)])
def test_a_prefix_of_a_longer_sequence(T, variants, split):
    import torch
    w = synth.CFG2.scaled(B=2, H=3, T=256, n_iter=6, seed=8800)
    x, g = synth.make_inputs(w), synth.make_gates(w)
    kw = dict(compute=binding.GKA_COMPUTE_BF16_SPLIT if split else binding.GKA_COMPUTE_BF16, path=binding.GKA_PATH_FUSED, walk_chunks=4)

    def forward(n):
        y = {m: np.ascontiguousarray(a[:, :n]) for m, a in {**x, **g}.items()}
        dev = upload_inputs(y, "bf16")
        opt = {m: to_device(y[m], "f32") for m in ("beta", "alpha")} if variants else {}
        o, ex = binding.gka_forward(*(dev[m] for m in ("q", "k", "v", "gate", "lam")), w.n_iter, return_fro=True, **kw, **opt)
        return o, ex["fro"]

    print("prefix", T, variants, split, flush=True)
    (o, fro), (oo, ff) = forward(T), forward(256)
    torch.cuda.synchronize()
    assert bool((o == oo[:, :T]).all()) and bool((fro == ff[:, :T]).all())


@pytest.mark.parametrize("T", [64, 129, 192, 320])
def test_states_after_an_odd_number_of_chunks(T):
    """U is not advanced over a second chunk that does not exist: the states of a walk of one chunk pair at a time, each of whose
    segments starts from summaries, and of the two-phase kernels."""
    import torch
    w = synth.CFG2.scaled(B=2, H=3, T=T, n_iter=4, seed=8900 + T)
    dev = upload_inputs(synth.make_inputs(w), "bf16")
    got = {}
    for name, kw in (("fused", dict(path=binding.GKA_PATH_FUSED, walk_chunks=64)), ("two-phase", dict(path=binding.GKA_PATH_TWO_PHASE))):
        got[name] = binding.gka_forward(*(dev[m] for m in ("q", "k", "v", "gate", "lam")), w.n_iter, return_state=True, **kw)[1]
    torch.cuda.synchronize()
    for n in ("H_final", "U_final"):                 # rows weighted and rounded to bf16 on both paths: 2^-9 of the terms of a sum
        a, b = got["fused"][n], got["two-phase"][n]
        assert float((a - b).norm() / b.norm()) <= 2.0 ** -8, n
