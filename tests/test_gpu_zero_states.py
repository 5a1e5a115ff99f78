"""Token by token from zero initial states where U is streamed through memory (d = 256; d = 128 for one token of many pairs):
whatever the final states' buffers and the workspace held before, here NaN, the results are the oracle's."""
import numpy as np
import pytest

import oracle
from paper_2511_21016_amd import binding, synth
from gka_testutil import to_device, to_host

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("final", [False, True])
@pytest.mark.parametrize("d,pairs,T", [(256, 3, 1), (256, 3, 2), (256, 260, 1), (256, 2, 5), (128, 300, 1), (128, 3, 1)])
def test_zero_states(d, pairs, T, final):
    import torch
    w = synth.CFG2.scaled(d=d, B=pairs, H=1, T=T, n_iter=4, seed=9900 + d + pairs + T)
    x = synth.make_inputs(w)
    dev = {n: to_device(x[n], "bf16" if n in "qkv" else "f32") for n in ("q", "k", "v", "gate", "lam")}
    params = binding.make_params(pairs, 1, T, d, w.n_iter, binding.GKA_BF16, binding.GKA_COMPUTE_BF16,
                                 path=binding.GKA_PATH_RECURRENT)
    nan = lambda *shape: torch.full(shape, float("nan"), device="cuda")
    nbytes = binding.forward_workspace_bytes(params)
    ws, o = nan(nbytes // 4), torch.full_like(dev["v"], float("nan"))
    H, U = nan(pairs, 1, d, d), nan(pairs, 1, d, d)
    ptr = lambda t: t.data_ptr()
    print("zero states", d, pairs, T, final, flush=True)
    st = binding.forward_raw(params, *(ptr(dev[n]) for n in ("q", "k", "v", "gate", "lam")), ptr(o), None, None,
                             ptr(H) if final else None, ptr(U) if final else None, None, ptr(ws), nbytes,
                             torch.cuda.current_stream().cuda_stream)
    assert st == binding.GKA_OK, binding.status_string(st)
    torch.cuda.synchronize()
    some = [0, pairs // 2, pairs - 1]
    ref, ex = oracle.forward(*(np.ascontiguousarray(x[n][some]) for n in ("q", "k", "v", "gate", "lam")), w.n_iter,
                             return_state=True)
    # float32 arithmetic, the outputs rounded to bf16 at 2^-9 of a value
    assert np.abs(to_host(o[some]) - ref).max() <= (1e-4 + 2.0 ** -8) * np.abs(ref).max()
    assert torch.isfinite(o.float()).all()
    if final:
        for got, name in ((H, "H_final"), (U, "U_final")):
            assert np.abs(to_host(got[some]) - ex[name]).max() <= 1e-6 * np.abs(ex[name]).max(), name
