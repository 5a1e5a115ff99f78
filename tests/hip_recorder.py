"""Runs calls of libgka in a child process whose HIP runtime is tests/hip_recorder.c: nothing is launched, and the kernels
that would have been, with their grids, come back. For tests of launch plans on the CPU."""
import os
import re
import subprocess
import sys
import tempfile

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)

VARIABLE = 1 << 60            # address of every device variable

# (the binding asks torch for its dtypes and the stream query only; torch itself would find the recorder for a runtime)
_PRELUDE = """
import ctypes, sys, types
sys.path.insert(0, {root!r})
torch = types.ModuleType("torch")
torch._C = types.SimpleNamespace(_cuda_getCurrentRawStream=lambda index: 0)
torch.float32, torch.bfloat16 = "float32", "bfloat16"
sys.modules["torch"] = torch
from paper_2511_21016_amd import binding
binding.load_library()
recorder = ctypes.CDLL({recorder!r})
set_device = recorder.recorder_set_device
recorder.recorder_words({words})
recorder.recorder_open({out!r}.encode())
"""


def kernel_name(mangled):
    """reverse_kernel from _ZN3gka14reverse_kernelI...: the identifier with "kernel" in it."""
    for m in re.finditer(r"\d+", mangled):
        name = mangled[m.end():m.end() + int(m.group())]
        if "kernel" in name:
            return name
    return mangled


def record(body, words=0):
    """Executes the source `body` with `binding` and `set_device` in scope. Returns the recorded calls as dicts; with `words`,
    launches have the first so many 8-byte words of their argument in "words"."""
    from paper_2511_21016_amd import binding, build
    if not os.path.exists(binding.LIB_PATH):
        build.build_library(verbose=False)
    with tempfile.TemporaryDirectory() as tmp:
        recorder, out = os.path.join(tmp, "hip_recorder.so"), os.path.join(tmp, "calls")
        subprocess.run(["gcc", "-O1", "-shared", "-fPIC", "-o", recorder, os.path.join(HERE, "hip_recorder.c")], check=True)
        source = _PRELUDE.format(root=ROOT, recorder=recorder, out=out, words=words) + body + "\nrecorder.recorder_close()\n"
        env = dict(os.environ)
        env["LD_PRELOAD"] = (recorder + " " + env.get("LD_PRELOAD", "")).strip()
        pr = subprocess.run([sys.executable, "-c", source], env=env, stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True,
                            timeout=120)
        assert pr.returncode == 0, pr.stdout
        calls = []
        for line in open(out):
            if line.startswith("words"):
                calls[-1]["words"] = [int(x) for x in line.split()[1:]]
                continue
            kind, name, a, b, c = line.split()
            call = {"kind": kind, "kernel": kernel_name(name), "mangled": name}
            if kind == "launch":
                call.update(grid=int(a), block=int(b), lds=int(c))
            elif kind == "variable":
                call.update(bytes=int(a))
            else:
                call.update(value=int(b), device=int(c))
            calls.append(call)
        return calls
