"""d = 16 and 32 with packed rows so wide (2^23 heads and more) that a tile of 16 tokens spans more than 4 GiB: the walk's lane
offsets are 64 bits wide there. Which kernel runs, on the CPU; results against the token-by-token path on the GPU."""
import pytest

from hip_recorder import record


@pytest.mark.parametrize("d,H,far", [(16, 1 << 16, False), (16, 8947848, False), (16, 8947849, True), (32, 4473923, False),
                                     (32, 4473925, True), (16, 1 << 24, True)])
def test_kernel_choice(d, H, far):
    calls = record(f"""
p = binding.make_params(1, {H}, 17, {d}, 5, binding.GKA_BF16, binding.GKA_COMPUTE_BF16)
X = 1 << 40
st = binding.forward_raw(p, X, X + 1, X + 2, X, X, X + 3, workspace=X, workspace_bytes=1 << 50)
assert st == binding.GKA_OK, binding.status_string(st)
""")
    walk = calls[-1]
    assert walk["kernel"] == "small_walk_kernel"
    # (the last template argument: WALK_NEAR, WALK_FAR; rows of the tile are up to 15 H d elements of 2 bytes away, features
    # up to 64 bytes)
    assert walk["mangled"].split("EEE")[0].endswith("Li1" if far else "Li0")
    assert far == (2 * (15 * H * d + 32) > 0xffffffff)


@pytest.mark.gpu
def test_against_the_token_by_token_path():
    import torch
    from paper_2511_21016_amd import binding
    H, T, d = (9 << 20) + 3, 17, 16                  # 4.8 GB per tensor, 39 GB of workspace
    torch.manual_seed(41)
    row = lambda: torch.randn(1, T, H, d, device="cuda", dtype=torch.bfloat16)
    q, k, v = row(), row(), row()
    k.mul_(0.25)
    gate = torch.rand(1, T, H, device="cuda")
    lam = torch.rand(1, T, H, device="cuda").add_(0.5)
    print("far rows", H, T, d, flush=True)
    o = binding.gka_forward(q, k, v, gate, lam, 4)
    ref = binding.gka_forward(q, k, v, gate, lam, 4, path=binding.GKA_PATH_RECURRENT)
    torch.cuda.synchronize()
    for t in range(T):                               # the stated bf16 tolerance, over a token's heads (2-norm: a few 1e-3)
        diff = (o[0, t].float() - ref[0, t].float()).norm() / ref[0, t].float().norm()
        assert float(diff) <= 2e-2, t
