"""gka_forward_static's fixed array: any problem of up to 341 (sequence, head) pairs fits, the launches' scratch ends within the
array, and a walk length that the caller asks for is kept and refused only where it takes more than 341 workgroups."""
import pytest

from hip_recorder import VARIABLE, record
from paper_2511_21016_amd import binding

MOST = 341                    # workgroups: GKA_STATIC_SCRATCH_BYTES / 196,612
SIZES = [(1, 16, 4096), (4, 16, 4096), (1, 32, 32768), (16, 16, 4096), (2, 8, 8192), (1, 1, 64), (1, 1, 1 << 20), (1, 16, 1337), (3, 12, 700),
         (128, 1, 500), (256, 1, 64), (256, 1, 2000), (11, 31, 64), (11, 31, 4096), (10, 20, 4096), (1, 342, 64), (64, 16, 1000)]


@pytest.mark.parametrize("compute", ["GKA_COMPUTE_BF16", "GKA_COMPUTE_BF16_SPLIT"])
@pytest.mark.parametrize("walk", [0, 1, 2, 7, 64, 2 ** 31 - 1])
def test_sizes(compute, walk):
    calls = record(f"""
for i, (B, H, T) in enumerate({SIZES}):
    p = binding.make_params(B, H, T, 128, 10, binding.GKA_BF16, binding.{compute}, walk_chunks={walk})
    a = [(i + 1 << 40) + (n << 36) for n in range(6)]
    st = binding.forward_static_raw(p, *a)
    most = {walk} if {walk} and {walk} < T // 64 + 1 else T // 64 + 1
    most += most % 2 if p.compute == binding.GKA_COMPUTE_BF16 else 0
    segs = ((T + 63) // 64 + most - 1) // most if {walk} else 1
    want = binding.GKA_OK if B * H * segs <= {MOST} else binding.GKA_ERR_STATIC_SCRATCH
    assert st == want, (B, H, T, binding.status_string(st))
""", words=32)
    array, = [c["bytes"] for c in calls if c["kind"] == "variable"]
    parked = 128 * 128 * 4 * (2 if compute.endswith("SPLIT") else 1)            # of a workgroup: U (and H)
    walks = [c for c in calls if c["kind"] == "launch" and c["kernel"] == "fused_forward_kernel"]
    assert walks
    for c in walks:
        assert c["grid"] <= MOST
        last = max(x for x in c["words"] if VARIABLE <= x < VARIABLE + (1 << 40))
        assert last - VARIABLE + c["grid"] * parked <= array


@pytest.mark.gpu
@pytest.mark.parametrize("B,H,T,walk,split", [(1, 16, 1337, 1, True), (11, 31, 130, 4, True), (11, 31, 130, 4, False), (1, 16, 1337, 0, True),
                                              (4, 16, 700, 0, False)])
def test_against_gka_forward(B, H, T, walk, split):
    """336 and 341 workgroups, with split operands beyond GKA_STATIC_SCRATCH_BYTES: the bits of gka_forward with the same walk.
    With a walk of the library's choice the start states may be composed in another order."""
    import torch
    from paper_2511_21016_amd import synth
    from gka_testutil import pair_rel_err, to_host, upload_inputs
    w = synth.CFG2.scaled(B=B, H=H, T=T, n_iter=6, seed=8100 + T)
    dev = upload_inputs(synth.make_inputs(w), w.dtype)
    compute = binding.GKA_COMPUTE_BF16_SPLIT if split else binding.GKA_COMPUTE_BF16
    args = [dev[n] for n in ("q", "k", "v", "gate", "lam")]
    print("static scratch", B, H, T, walk, split, flush=True)
    want = binding.gka_forward(*args, w.n_iter, compute=compute, walk_chunks=walk)
    o = torch.full_like(dev["v"], float("nan"))
    p = binding.make_params(B, H, T, 128, w.n_iter, binding.GKA_BF16, compute, walk_chunks=walk)
    st = binding.forward_static_raw(p, *(t.data_ptr() for t in args), o.data_ptr(), stream=torch.cuda.current_stream().cuda_stream)
    assert st == binding.GKA_OK, binding.status_string(st)
    torch.cuda.synchronize()
    if walk:
        assert torch.equal(o, want)
    # (float32 states that differ in their last bits, rounded to bf16: less than the 2e-2 that either side is allowed)
    assert pair_rel_err(to_host(o), to_host(want)) <= 1e-2
