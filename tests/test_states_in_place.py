"""gka_forward whose final states go to the buffers of its initial ones (a sequence continued in place). At d = 16, 32 and 256
every shape takes such a call: no wave may still have to read an initial state when another one writes the final state over
it. Launch plans, on the CPU: which kernels would run, and in how many workgroups."""
import pytest

from hip_recorder import record

_CALL = """
H, U, X = 0x10000000, 0x20000000, 0x30000000
p = binding.make_params({B}, {heads}, {T}, {d}, 5, binding.{io}, binding.{compute})
st = binding.forward_raw(p, X, X + 0x1000000, X + 0x2000000, X, X, X + 0x3000000, H, U, {final}, None, 0x40000000, 1 << 42)
assert st == binding.GKA_OK, binding.status_string(st)
"""


def _launches(d, B, heads, T, io, compute, in_place):
    final = "H, U" if in_place else "H + 0x8000000, U + 0x8000000"
    return [c for c in record(_CALL.format(d=d, B=B, heads=heads, T=T, io=io, compute=compute, final=final))
            if c["kind"] == "launch"]


@pytest.mark.parametrize("d,B,H,T", [(16, 2, 3, 1), (16, 2, 3, 128), (32, 1, 2, 128), (16, 4, 6, 197), (32, 2, 3, 250),
                                     (16, 16, 12, 250), (16, 16, 12, 705), (16, 41, 25, 65), (32, 64, 16, 129)])
def test_small_head_dims(d, B, H, T):
    plan = _launches(d, B, H, T, "GKA_BF16", "GKA_COMPUTE_BF16", True)
    names = [c["kernel"] for c in plan]
    if "small_state_scan_kernel" in names:           # one thread reads and writes an element, ahead of the walk
        assert names.index("small_state_scan_kernel") == len(names) - 2
    else:                                            # one wave per pair reads its states first and writes them last
        assert names == ["small_walk_kernel"] and plan[0]["grid"] == (B * H + 3) // 4


@pytest.mark.parametrize("B,H,T,io,compute", [(1, 2, 129, "GKA_F32", "GKA_COMPUTE_F32"),
                                              (2, 3, 400, "GKA_BF16", "GKA_COMPUTE_BF16"),
                                              (1, 1, 4096, "GKA_BF16", "GKA_COMPUTE_F32")])
def test_head_dim_256(B, H, T, io, compute):
    # one segment: the workgroups of the state pass (8 slabs of H, 8 of U per pair) are all there are
    passes = lambda in_place: [c["grid"] for c in _launches(256, B, H, T, io, compute, in_place)
                               if c["kernel"] == "state_pass_kernel"]
    assert passes(True) == [B * H * 16]
    if T > 64 * 5:                                   # (separate buffers are cut into segments: a summary launch before it)
        assert len(passes(False)) == 2


@pytest.mark.gpu
@pytest.mark.parametrize("d,B,H,T", [(16, 2, 3, 40), (32, 1, 3, 64), (16, 2, 3, 128), (16, 4, 6, 197), (32, 2, 3, 250),
                                     (16, 41, 25, 65), (256, 1, 2, 145), (256, 2, 3, 400)])
def test_in_place_against_separate_buffers(d, B, H, T):
    import numpy as np
    import torch
    import oracle
    from paper_2511_21016_amd import binding, synth
    from gka_testutil import pair_rel_err, to_device, to_host, upload_inputs
    w = synth.CFG2.scaled(d=d, B=B, H=H, T=T, n_iter=5, seed=5200 + d + T)
    x = synth.make_inputs(w)
    rng = np.random.default_rng(w.seed)
    A = rng.standard_normal((B, H, d, 8)) / np.sqrt(d)
    H0, U0 = (A @ np.transpose(A, (0, 1, 3, 2))).astype(np.float32), (rng.standard_normal((B, H, d, d)) / d).astype(np.float32)
    dev, Hs, Us = upload_inputs(x, "bf16"), to_device(H0, "f32"), to_device(U0, "f32")
    params = binding.make_params(B, H, T, d, w.n_iter, binding.GKA_BF16, binding.GKA_COMPUTE_BF16)
    nbytes = binding.forward_workspace_bytes(params)
    ws, o = torch.empty(nbytes, dtype=torch.uint8, device="cuda"), torch.empty_like(dev["v"])
    print("in place", d, B, H, T, flush=True)
    st = binding.forward_raw(params, *(dev[n].data_ptr() for n in ("q", "k", "v", "gate", "lam")), o.data_ptr(),
                             Hs.data_ptr(), Us.data_ptr(), Hs.data_ptr(), Us.data_ptr(), None, ws.data_ptr(), nbytes,
                             torch.cuda.current_stream().cuda_stream)
    assert st == binding.GKA_OK, binding.status_string(st)
    torch.cuda.synchronize()
    ref, ex = oracle.forward(x["q"], x["k"], x["v"], x["gate"], x["lam"], w.n_iter, H_init=H0, U_init=U0, return_state=True)
    # the stated bf16 tolerance; the states at d = 256 are float32 sums, at 16 and 32 sums of rounded outer products
    assert pair_rel_err(to_host(o), ref) <= 2e-2
    for got, name in ((Hs, "H_final"), (Us, "U_final")):
        assert np.abs(to_host(got) - ex[name]).max() <= (1e-5 if d == 256 else 5e-3) * np.abs(ex[name]).max(), name
