"""The segments of the fused kernels' chunk walk: chosen for the number of workgroups that they make. The workspace size, which
bounds them, does not shrink with the problem or depend on the passes; results do not depend on the choice."""
import itertools

import pytest

import oracle
from paper_2511_21016_amd import binding, synth
from gka_testutil import pair_rel_err, to_host, upload_inputs

FUSED = binding.GKA_PATH_FUSED
SPLIT = binding.GKA_COMPUTE_BF16_SPLIT


def nbytes(pairs, T, n_iter=10, compute=binding.GKA_COMPUTE_BF16, path=FUSED):
    return binding.forward_workspace_bytes(binding.make_params(1, pairs, T, 128, n_iter, binding.GKA_BF16, compute, path=path))


@pytest.mark.parametrize("compute,path", [(binding.GKA_COMPUTE_BF16, FUSED), (SPLIT, binding.GKA_PATH_AUTO)])
def test_a_workspace_serves_every_smaller_call(compute, path):
    sizes = {(P, T): nbytes(P, T, 10, compute, path)
             for P, T in itertools.product((1, 4, 36, 48, 100, 200, 256, 300, 512, 1025), (1, 64, 65, 300, 1337, 2000, 4096, 20000))}
    for (P, T), (Q, U) in itertools.product(sizes, sizes):
        if P <= Q and T <= U:
            assert sizes[P, T] <= sizes[Q, U]
    for (P, T), n in sizes.items():
        assert n == nbytes(P, T, 0, compute, path) == nbytes(P, T, 30, compute, path)


@pytest.mark.gpu
@pytest.mark.parametrize("B,H,T,compute", [(3, 12, 700, binding.GKA_COMPUTE_BF16),      # 36 pairs, 11 chunks: 6 segments
                                           (5, 20, 450, binding.GKA_COMPUTE_BF16),      # 100 pairs, 8 chunks: 2
                                           (10, 30, 390, binding.GKA_COMPUTE_BF16),     # 300 pairs, 7 chunks: several rounds
                                           (3, 12, 450, SPLIT)])
def test_segments_against_one_walk(B, H, T, compute):
    import torch
    w = synth.CFG2.scaled(B=B, H=H, T=T, seed=77 + H)
    x = synth.make_inputs(w)
    dev = upload_inputs(x, w.dtype)
    args = (dev["q"], dev["k"], dev["v"], dev["gate"], dev["lam"], w.n_iter)
    # (a workspace full of NaN: nothing may be read from it that has not been written)
    ws = torch.full((nbytes(B * H, T, 10, compute) // 4 + 64,), float("nan"), device="cuda")
    ws = ws.view(torch.uint8)[:nbytes(B * H, T, 10, compute)]
    o, ex = binding.gka_forward(*args, compute=compute, path=FUSED, return_state=True, workspace=ws)
    one, eo = binding.gka_forward(*args, compute=compute, path=FUSED, return_state=True, walk_chunks=(T + 63) // 64 + 1)
    torch.cuda.synchronize()
    # float32 states composed in another order differ in their last bits, which the rounding of H_[n] to bf16 turns into
    # steps of 2^-9 of single elements now and then: far less than the 2e-2 that both sides are allowed
    assert pair_rel_err(to_host(o), to_host(one)) <= 1e-2
    for name in ("H_final", "U_final"):
        a, b = to_host(ex[name]), to_host(eo[name])
        assert abs(a - b).max() <= 2e-3 * abs(b).max()
    ref = oracle.forward(x["q"][:1], x["k"][:1], x["v"][:1], x["gate"][:1], x["lam"][:1], w.n_iter)
    assert pair_rel_err(to_host(o[:1]), ref) <= 2e-2
