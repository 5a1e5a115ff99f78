"""Kernels with more dynamic LDS than a launch has by default (64 KiB): their limit is an attribute of the kernel on one
device, so a process that uses a second GPU has to raise it there as well. On the CPU, with two devices pretended."""
import pytest

from hip_recorder import record

DEFAULT_LDS = 64 << 10

_CALLS = {
    "forward": "binding.forward_raw(p, X, X + 1, X + 2, X, {lam}, X + 3, workspace=X, workspace_bytes=1 << 42)",
    "backward": "binding.backward_raw(p, X, X, X, X, {lam}, X, X, X, X, X, workspace=X, workspace_bytes=1 << 42)",
    "sketched": "binding.forward_sketched_raw(p, X, X, X, X, {lam}, X, 32, 0, X, workspace=X, workspace_bytes=1 << 42)",
}


_SHAPES = [(64, "bf16", False), (64, "bf16", True), (128, "bf16", False), (128, "bf16", True), (64, "f32", False),
           (128, "f32", True), (256, "f32", False)]


@pytest.mark.parametrize("call,d,dtype,variants", [
    (call, *shape) for call in sorted(_CALLS) for shape in _SHAPES
    if shape[0] < 256 or call == "forward" if call != "sketched" or shape[1:] == ("bf16", False)])
def test_limits_are_raised_on_every_device(call, d, dtype, variants):
    io, compute = {"f32": ("GKA_F32", "GKA_COMPUTE_F32"), "bf16": ("GKA_BF16", "GKA_COMPUTE_BF16")}[dtype]
    opts = "lambda_scale=0.05, beta=1 << 30, alpha=1 << 30" if variants else ""
    calls = record(f"""
X = 0x10000000
p = binding.make_params(2, 3, 400, {d}, 5, binding.{io}, binding.{compute}, {opts})
for device in (0, 1):
    set_device(device)
    st = {_CALLS[call].format(lam="None" if variants else "X")}
    assert st == binding.GKA_OK, binding.status_string(st)
""")
    raised, device, launches = {}, 0, 0
    half = sum(c["kind"] == "launch" for c in calls) // 2      # the first half of the launches is the first device's
    for c in calls:
        if c["kind"] == "attribute":
            raised[c["mangled"], c["device"]] = c["value"]
            continue
        device, launches = int(launches >= half), launches + 1
        if c["lds"] > DEFAULT_LDS:
            assert raised.get((c["mangled"], device), 0) >= c["lds"], (c["kernel"], device)
