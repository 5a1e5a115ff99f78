"""d = 256 chunk-wise: the bound of its workspace (512 KiB of chunk states per pair and chunk, 1 GiB in all) and, on the GPU,
problems that it cuts into several batches of pairs and slabs of chunks, against the fp64 oracle."""
import numpy as np
import pytest

from paper_2511_21016_amd import binding

GIB = 1 << 30


@pytest.mark.parametrize("B,H", [(1, 1), (4, 8), (64, 8), (128, 8), (700, 8)])
@pytest.mark.parametrize("T", [129, 192, 256, 257, 1024, 65536])
def test_workspace_bound(B, H, T):
    p = binding.make_params(B, H, T, 256, 10, binding.GKA_BF16, binding.GKA_COMPUTE_BF16)
    total = binding.forward_workspace_bytes(p)
    chunks = (T + 63) // 64
    pairs = min(B * H, 2048 // min(chunks, 4))              # pairs of a launch: at least four chunks of each fit
    carried = pairs << 20 if pairs * chunks > 2048 else 0   # two (H, U) pairs, where the sequence takes several slabs
    assert 0 < total <= GIB + carried + (64 << 20)          # (64 MiB: norms, summaries of up to some 32 segments)


@pytest.mark.parametrize("budget", [1, 4 << 20, 64 << 20])
def test_workspace_follows_the_callers_budget(budget):
    p = binding.make_params(3, 7, 1000, 256, 10, binding.GKA_F32, binding.GKA_COMPUTE_F32, slab_state_bytes=budget)
    states = max(budget, 4 * (512 << 10))                   # one pair's four chunks at least
    pairs = states // (4 * (512 << 10))
    # summaries: 32 segments of 512 KiB at most (16 workgroups per segment and pair, 256 wanted)
    assert binding.forward_workspace_bytes(p) <= states + (min(pairs, 21) << 20) + (32 << 19) + (1 << 20)


def _inputs(w):
    from paper_2511_21016_amd import synth
    x = synth.make_inputs(w)
    g = synth.make_gates(w)
    rng = np.random.default_rng(w.seed)
    A = rng.standard_normal((w.B, w.H, 256, 8)) / 16.0
    return x, dict(beta=g["beta"], alpha=g["alpha"], H_init=(A @ np.transpose(A, (0, 1, 3, 2))).astype(np.float32),
                   U_init=(rng.standard_normal((w.B, w.H, 256, 256)) / 256).astype(np.float32))


@pytest.mark.gpu
@pytest.mark.parametrize("dtype,budget", [("f32", 4 << 20), ("bf16", 1), ("f32", 24 << 20)])
def test_batches_and_slabs(dtype, budget):
    # 5 pairs x 13 chunks: batches of 2, 1 and 5 pairs, slabs of 4, 4 and 9 chunks
    import torch
    import oracle
    from paper_2511_21016_amd import synth
    from gka_testutil import pair_rel_err, to_device, to_host, upload_inputs
    w = (synth.CFG2 if dtype == "bf16" else synth.CFG1).scaled(d=256, B=5, H=1, T=777, n_iter=5, seed=9300 + budget % 97)
    x, opt = _inputs(w)
    dev = upload_inputs(x, dtype)
    print("wide slabs", dtype, budget, flush=True)
    o, ex = binding.gka_forward(dev["q"], dev["k"], dev["v"], dev["gate"], dev["lam"], w.n_iter, return_state=True,
                                return_fro=True, slab_state_bytes=budget,
                                compute=binding.GKA_COMPUTE_F32, **{n: to_device(a, "f32") for n, a in opt.items()})
    torch.cuda.synchronize()
    ref, rex = oracle.forward(x["q"], x["k"], x["v"], x["gate"], x["lam"], w.n_iter, return_state=True, return_fro=True, **opt)
    # float32 sums (1e-4, the bound of every float32 path); bf16 outputs round at 2^-9 of a value
    assert pair_rel_err(to_host(o), ref) <= (1e-4 if dtype == "f32" else 1e-4 + 2.0 ** -8)
    assert np.abs(to_host(ex["fro"]) - rex["fro"]).max() <= 1e-5 * rex["fro"].max()
    for n in ("H_final", "U_final"):
        assert np.abs(to_host(ex[n]) - rex[n]).max() <= 1e-5 * np.abs(rex[n]).max(), n


@pytest.mark.gpu
def test_more_pairs_than_a_launch_takes():
    # 1400 pairs x 3 chunks: batches of 682 pairs; the pairs at the edges of the batches
    import torch
    import oracle
    from paper_2511_21016_amd import synth
    from gka_testutil import pair_rel_err, to_host, upload_inputs
    w = synth.CFG2.scaled(d=256, B=1400, H=1, T=130, n_iter=3, seed=9399)
    x = synth.make_inputs(w)
    dev = upload_inputs(x, "bf16")
    print("wide pairs", flush=True)
    o, ex = binding.gka_forward(dev["q"], dev["k"], dev["v"], dev["gate"], dev["lam"], w.n_iter, return_state=True)
    torch.cuda.synchronize()
    some = [0, 681, 682, 1363, 1364, 1399]
    ref, rex = oracle.forward(*(np.ascontiguousarray(x[n][some]) for n in ("q", "k", "v", "gate", "lam")), w.n_iter,
                              return_state=True)
    assert pair_rel_err(to_host(o[some]), ref) <= 1e-4 + 2.0 ** -8
    for n in ("H_final", "U_final"):
        assert np.abs(to_host(ex[n][some]) - rex[n]).max() <= 1e-5 * np.abs(rex[n]).max(), n
