"""The backward pass's workspace: what the query asks for (only the tensors that a dtype's path uses), and that a pass keeps
within it and takes nothing from what it held before."""
import pytest

from hip_recorder import record
from paper_2511_21016_amd import binding

STATE_BYTES = 128 * 128 * 4


@pytest.mark.parametrize("dtype,d", [("bf16", 64), ("bf16", 128), ("f32", 64), ("f32", 128)])
def test_query(dtype, d):
    B, H, T = 3, 8, 700
    io, compute = (binding.GKA_BF16, binding.GKA_COMPUTE_BF16) if dtype == "bf16" else (binding.GKA_F32, binding.GKA_COMPUTE_F32)
    p = binding.make_params(B, H, T, d, 10, io, compute)
    tensor = B * T * H * d * (2 if dtype == "bf16" else 4)
    # besides the tensors: nine scalars per token, three states per pair, the scratch of the passes (the forward workspace with the
    # more numerous segments of the plain readouts, or the segment summaries of the readouts and the reverse walk)
    scalars, states, chunks = 9 * 4 * B * T * H, 3 * 4 * B * H * d * d, B * H * ((T + 63) // 64)
    scratch = chunks * (3 * d * d * 4 + 4096) + (1 << 20)
    total = binding.backward_workspace_bytes(p)
    assert total <= (17 if dtype == "bf16" else 23) * tensor + scalars + states + scratch


PAIRS = ((1, 1), (1, 4), (2, 3), (3, 16), (5, 20), (8, 32), (10, 30), (16, 32), (19, 31), (24, 32), (32, 32), (41, 25), (33, 32),
         (48, 32), (64, 32), (128, 24), (128, 32))
CHUNKS = (1, 2, 3, 4, 5, 6, 7, 8, 9, 11, 15, 16, 17, 23, 32, 39, 63, 64, 65, 129)


@pytest.mark.parametrize("n_iter,walk_chunks", [(0, 0), (10, 0), (40, 0), (10, 1), (10, 5), (10, 2 ** 31 - 1)])
def test_the_solves_walk_keeps_within_it(n_iter, walk_chunks):
    """From the arguments of the launches: the blocks in which the workgroups of the solves' walk park their states and vectors, the
    last thing in the workspace, end within what the query asked for, and the query does not depend on the passes."""
    cases = [(B, H, 64 * n - n % 2) for B, H in PAIRS for n in CHUNKS if n > 1 or B * H <= 256]      # (else no walk)
    calls = record(f"""
for i, (B, H, T) in enumerate({cases}):
    p = binding.make_params(B, H, T, 128, {n_iter}, binding.GKA_BF16, binding.GKA_COMPUTE_BF16, walk_chunks={walk_chunks})
    q, k, v, gate, lam, dy, dq, dk, dv, dgate = (n << 32 for n in range(1, 11))
    W, size = (i + 1) << 44, binding.backward_workspace_bytes(p)
    assert size < 1 << 44
    st = binding.backward_raw(p, q, k, v, gate, lam, dy, dq, dk, dv, dgate, dlam=dq, workspace=W, workspace_bytes=size)
    assert st == binding.GKA_OK, binding.status_string(st)
""", words=48)
    walks = [c for c in calls if c["kind"] == "launch" and c["kernel"] == "dual_solve_kernel"]
    assert len(walks) == len(cases)
    for i, (B, H, T) in enumerate(cases):
        size = binding.backward_workspace_bytes(binding.make_params(B, H, T, 128, 10, binding.GKA_BF16, binding.GKA_COMPUTE_BF16,
                                                                    walk_chunks=walk_chunks))
        W, walk = (i + 1) << 44, walks[i]
        assert 0 < walk["grid"] <= max(1024, B * H) or walk_chunks
        parked = max(x for x in walk["words"] if W <= x < W + (1 << 44))
        assert parked - W + walk["grid"] * 2 * STATE_BYTES <= size, (B, H, T, walk["grid"])


@pytest.mark.gpu
@pytest.mark.parametrize("dtype,d,opts", [("bf16", 128, ()), ("bf16", 64, ("alpha", "beta")), ("bf16", 128, ("alpha", "rule")),
                                          ("bf16", 64, ("rule", "state")), ("f32", 64, ("alpha", "rule")), ("f32", 128, ())])
def test_pass_keeps_within_it(dtype, d, opts):
    import torch
    B, H, T, r = 2, 3, 333, 5
    dt = torch.bfloat16 if dtype == "bf16" else torch.float32
    g = torch.Generator(device="cuda").manual_seed(17 + d)
    normal = lambda *s: torch.randn(s, generator=g, device="cuda")
    row = lambda: torch.nn.functional.normalize(normal(B, T, H, d), dim=-1).to(dt)
    q, k, v, dy = row(), row(), normal(B, T, H, d).to(dt), normal(B, T, H, d).to(dt)
    gate = torch.sigmoid(normal(B, T, H) + 3.0)
    lam = None if "rule" in opts else torch.nn.functional.softplus(normal(B, T, H)) + 0.01
    kw = {n: torch.sigmoid(normal(B, T, H)) for n in ("alpha", "beta") if n in opts}
    if "rule" in opts:
        kw["lambda_scale"] = 0.05
    if "state" in opts:
        A = normal(B, H, d, d) * 0.05
        kw.update(H_init=(A @ A.transpose(-1, -2)).contiguous(), U_init=normal(B, H, d, d) * 0.05, return_state_grads=True)
    io, compute = (binding.GKA_BF16, binding.GKA_COMPUTE_BF16) if dtype == "bf16" else (binding.GKA_F32, binding.GKA_COMPUTE_F32)
    some = gate.data_ptr()
    p = binding.make_params(B, H, T, d, r, io, compute, lambda_scale=kw.get("lambda_scale", 0.0),
                            alpha=some if "alpha" in opts else None, beta=some if "beta" in opts else None)
    nbytes = binding.backward_workspace_bytes(p)
    results = []
    for fill in (0, 255):                            # (bytes of 255: NaN in bf16 and in float32)
        ws = torch.full((nbytes + 4096,), fill, dtype=torch.uint8, device="cuda")
        ws[nbytes:] = 77
        print("backward workspace", dtype, d, opts, fill, flush=True)
        results.append(binding.gka_backward(q, k, v, gate, lam, dy, r, workspace=ws[:nbytes], **kw))
        torch.cuda.synchronize()
        assert bool((ws[nbytes:] == 77).all())
    for name, a in results[0].items():
        assert torch.isfinite(a).all() and torch.equal(a, results[1][name]), name
