"""gka_forward whose outputs replace its values (o == v) or keys (o == k), where a workgroup or wave reads rows of a chunk that
others solve: float32 products, or those of 16-bit pieces at d = 256 (a chunk's token blocks in workgroups of their own), and d =
16 and 32 (waves that advance the states over tiles of other waves). Launch plans on the CPU, results on the GPU."""
import pytest

from hip_recorder import record

_CALL = """
Q, K, V, O, X, W = (n << 36 for n in range(1, 7))
p = binding.make_params({B}, {H}, {T}, {d}, {n_iter}, binding.{io}, binding.{compute})
st = binding.forward_raw(p, Q, K, V, X, X, {o}, workspace=W, workspace_bytes=1 << 42)
assert st == binding.GKA_OK, binding.status_string(st)
"""


def _launches(d, B, H, T, dtype, o, n_iter=5):
    io, compute = {"f32": ("GKA_F32", "GKA_COMPUTE_F32"), "bf16": ("GKA_BF16", "GKA_COMPUTE_BF16"),
                   "bf16, f32": ("GKA_BF16", "GKA_COMPUTE_F32")}[dtype]
    return [c for c in record(_CALL.format(d=d, B=B, H=H, T=T, io=io, compute=compute, o=o, n_iter=n_iter))
            if c["kind"] == "launch"]


@pytest.mark.parametrize("o", ["V", "K"])
@pytest.mark.parametrize("d,B,H,T,dtype,n_iter,blocks,kernel", [(64, 1, 2, 130, "f32", 5, 4, "solve_f32_kernel"),
                                                                (64, 4, 8, 500, "f32", 5, 2, "solve_f32_kernel"),
                                                                (128, 1, 3, 200, "f32", 5, 4, "solve_f32_kernel"),
                                                                (256, 1, 2, 300, "f32", 5, 4, "solve_f32_kernel"),
                                                                (256, 4, 8, 300, "f32", 5, 2, "solve_f32_kernel"),
                                                                (256, 1, 2, 300, "bf16, f32", 5, 4, "solve_f32_kernel"),
                                                                (256, 4, 8, 300, "bf16, f32", 5, 2, "solve_f32_kernel"),
                                                                (256, 1, 2, 300, "bf16", 5, 4, "solve_wide_kernel"),
                                                                (256, 4, 8, 300, "bf16", 60, 2, "solve_wide_kernel"),
                                                                (256, 1, 2, 300, "bf16", 61, 4, "solve_f32_kernel"),
                                                                (256, 4, 8, 300, "bf16", 61, 2, "solve_f32_kernel")])
def test_float32_products(d, B, H, T, dtype, n_iter, blocks, kernel, o):
    chunks = B * H * ((T + 63) // 64)

    def solves(dst):
        plan = [c for c in _launches(d, B, H, T, dtype, dst, n_iter) if c["kernel"].startswith("solve")]
        assert {c["kernel"] for c in plan} == {kernel}
        return [c["grid"] for c in plan]
    assert solves("O") == [chunks * blocks]
    assert solves(o) == [chunks] * blocks            # one token block of every chunk per launch


@pytest.mark.parametrize("o", ["V", "K"])
@pytest.mark.parametrize("d,B,H,T", [(16, 2, 3, 128), (16, 4, 6, 197), (32, 2, 3, 150), (32, 2, 3, 500), (16, 15, 12, 390)])
def test_small_head_dims(d, B, H, T, o):
    plan = _launches(d, B, H, T, "bf16", o)
    if plan[-1]["mangled"].split("EEE")[0].endswith("Li2"):    # WALK_CHUNK: a workgroup has read its chunk before it stores
        assert plan[-1]["grid"] == B * H * ((T + 63) // 64)
        return
    walks_per_pair = (T + 63) // 64 if "small_state_scan_kernel" in [c["kernel"] for c in plan] else 1
    assert plan[-1]["kernel"] == "small_walk_kernel" and plan[-1]["grid"] == (B * H * walks_per_pair + 3) // 4


@pytest.mark.gpu
@pytest.mark.parametrize("name", ["v", "k"])
@pytest.mark.parametrize("d,dtype,B,H,T", [(16, "bf16", 2, 3, 128), (32, "bf16", 2, 3, 300), (64, "f32", 2, 3, 150),
                                           (128, "f32", 3, 8, 600), (256, "bf16", 2, 3, 200)])
def test_in_place_against_separate_outputs(d, dtype, B, H, T, name):
    import torch
    from paper_2511_21016_amd import binding, synth
    from gka_testutil import pair_rel_err, to_host, upload_inputs
    w = (synth.CFG2 if dtype == "bf16" else synth.CFG1).scaled(d=d, B=B, H=H, T=T, n_iter=5, seed=8800 + d + T)
    dev = upload_inputs(synth.make_inputs(w), dtype)
    args = [dev[n] for n in ("q", "k", "v", "gate", "lam")]
    print("outputs in place", d, dtype, B, H, T, name, flush=True)
    want = to_host(binding.gka_forward(*args, w.n_iter))
    got = to_host(binding.gka_forward(*args, w.n_iter, out=dev[name]))
    # the same sums at float32 products; d = 16, 32: tiles solved against other (rounded) states, twice the rounding that the
    # outputs are allowed
    assert pair_rel_err(got, want) <= (0.0 if d >= 64 else 2e-2)


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
def test_gate_gradients_over_the_gates(dtype):
    """The gate gradient's scan reads gates across the ranges of its waves: with dgate == gate it has one wave."""
    call = """
ptr = [n << 36 for n in range(1, 12)]
p = binding.make_params(1, 2, 1000, 64, 5, binding.{io}, binding.{compute})
q, k, v, gate, lam, dy, dq, dk, dv, ws, dgate = ptr
st = binding.backward_raw(p, q, k, v, gate, lam, dy, dq, dk, dv, {dgate}, workspace=ws, workspace_bytes=1 << 42)
assert st == binding.GKA_OK, binding.status_string(st)
"""
    io, compute = {"f32": ("GKA_F32", "GKA_COMPUTE_F32"), "bf16": ("GKA_BF16", "GKA_COMPUTE_BF16")}[dtype]
    waves = lambda dgate: [c["block"] // 64 for c in record(call.format(io=io, compute=compute, dgate=dgate))
                           if c["kernel"] == "bwd_scan_kernel"]
    assert waves("dgate") == [16] and waves("gate") == [1]


@pytest.mark.gpu
def test_gate_gradients_over_the_gates_against_separate_ones():
    import torch
    from paper_2511_21016_amd import binding, synth
    from gka_testutil import to_host, upload_inputs
    w = synth.CFG1.scaled(B=1, H=2, T=1000, d=64, n_iter=5, seed=771)
    x = synth.make_inputs(w)
    x["gate"][0, 500, 1] = 0.0
    dev = upload_inputs(x, "f32")
    dy = torch.randn(dev["v"].shape, generator=torch.Generator(device="cuda").manual_seed(3), device="cuda")
    params = binding.make_params(1, 2, 1000, 64, w.n_iter, binding.GKA_F32, binding.GKA_COMPUTE_F32)
    nbytes = binding.backward_workspace_bytes(params)
    ws = torch.empty(nbytes, dtype=torch.uint8, device="cuda")
    grads = [torch.empty_like(dev["q"]) for _ in range(3)]
    results = []
    for in_place in (False, True):
        gate = dev["gate"].clone()
        dgate = gate if in_place else torch.empty_like(gate)
        st = binding.backward_raw(params, dev["q"].data_ptr(), dev["k"].data_ptr(), dev["v"].data_ptr(), gate.data_ptr(),
                                  dev["lam"].data_ptr(), dy.data_ptr(), *(g.data_ptr() for g in grads), dgate.data_ptr(),
                                  workspace=ws.data_ptr(), workspace_bytes=nbytes,
                                  stream=torch.cuda.current_stream().cuda_stream)
        assert st == binding.GKA_OK, binding.status_string(st)
        torch.cuda.synchronize()
        results.append(to_host(dgate))
    # float32 sums of 1000 terms in another order
    assert abs(results[1] - results[0]).max() <= 1e-4 * abs(results[0]).max()
