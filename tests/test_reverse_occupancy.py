"""The reverse walks of one recurrence each (with an alpha-connection) at d = 64: with more workgroups than compute units two of
them share one, so that a workgroup may take half of its LDS. Which variant is launched, on the CPU; gradients on the GPU."""
import numpy as np
import pytest

from hip_recorder import record

HALF_LDS = 80 << 10


@pytest.mark.parametrize("d,pairs,T,alpha,shared", [(64, 256, 300, True, False), (64, 257, 300, True, True), (64, 200, 1000, True, True),
                                                    (64, 100, 300, True, False), (64, 2000, 1, True, True),
                                                    (64, 300, 300, False, False), (128, 300, 300, True, False)])
def test_which_variant(d, pairs, T, alpha, shared):
    calls = record(f"""
p = binding.make_params(1, {pairs}, {T}, {d}, 5, binding.GKA_BF16, binding.GKA_COMPUTE_BF16, alpha=1 << 30 if {alpha} else None)
X = 1 << 40
st = binding.backward_raw(p, X, X, X, X, X, X, X, X, X, X, dlam=X, workspace=X, workspace_bytes=1 << 50)
assert st == binding.GKA_OK, binding.status_string(st)
""")
    walks = [c for c in calls if c["kind"] == "launch" and c["kernel"] == "reverse_kernel" and "Lb0ELb" in c["mangled"]]
    assert len(walks) == (2 if alpha else 1)
    for c in walks:
        assert c["grid"] >= pairs and (c["lds"] <= HALF_LDS) == shared, (c["grid"], c["lds"])


@pytest.mark.gpu
@pytest.mark.parametrize("T", [1, 64, 65, 190, 330])
def test_many_pairs_against_the_oracle(T):
    import torch
    from oracle import gka_backward_oracle as bwd
    from paper_2511_21016_amd import binding, synth
    from gka_testutil import to_device, to_host, upload_inputs
    w = synth.CFG2.scaled(B=2, H=3, T=T, d=64, n_iter=6, gate_mean=4.0, seed=9700 + T)
    x, g = synth.make_inputs(w), synth.make_gates(w)
    x["lam"] = (x["lam"] + 0.25).astype(np.float32)      # (condition numbers of 20 at most: the bound below is that of such systems)
    if T > 100:
        x["gate"][0, 77, 1] = 0.0                        # a packed sequence starts inside a chunk
    dy = synth.round_to_bf16(np.random.default_rng(w.seed).standard_normal(x["v"].shape).astype(np.float32))
    dev = upload_inputs(x, "bf16")
    many = [t.repeat(50, *[1] * (t.dim() - 1)).contiguous()
            for t in [dev[n] for n in ("q", "k", "v", "gate", "lam")] + [to_device(dy, "bf16")] + [to_device(g[n], "f32") for n in ("beta", "alpha")]]
    print("reverse walks of 300 pairs", T, flush=True)
    out = binding.gka_backward(*many[:6], w.n_iter, beta=many[6], alpha=many[7])
    torch.cuda.synchronize()
    ref = bwd.backward(x["q"], x["k"], x["v"], x["gate"], x["lam"], dy, w.n_iter, beta=g["beta"], alpha=g["alpha"])
    for n, a in out.items():
        a, want = to_host(a), ref[n].copy()
        assert all((a[i:i + 2] == a[:2]).all() for i in range(0, 100, 2)), n
        if n == "dgate":
            want[x["gate"] == 0.0] = 0.0                 # (reported as 0 at a gate of 0)
            if T == 1:                                   # (it multiplies a zero state)
                assert np.abs(a).max() <= 2e-3
                continue
        err = np.abs(a[:2] - want).max() / np.abs(want).max()
        print(n, err, flush=True)
        assert err <= 2e-2, (n, err)                     # the stated tolerance of the backward pass on bf16 operands
