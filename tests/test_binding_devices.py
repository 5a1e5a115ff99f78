"""The binding refuses tensors that are not on a GPU before it calls the library: a kernel given their addresses would fault.
CPU only: the library's entry points are replaced, so that nothing can be launched whatever the binding does."""
import pytest
import torch

from paper_2511_21016_amd import binding

B, T, H, D = 2, 3, 2, 64


@pytest.fixture
def no_launch(monkeypatch):
    binding.load_library()
    calls = []
    for name in ("forward_raw", "decode_step_raw", "decode_tokens_raw", "backward_raw", "backward_from_state_raw",
                 "forward_sketched_raw"):
        monkeypatch.setattr(binding, name, lambda *a, _name=name, **kw: calls.append(_name) or binding.GKA_OK)
    monkeypatch.setattr(binding, "_raw_stream", lambda index: 0)
    return calls


def _args(*lead):
    bf16 = lambda: torch.zeros(*lead, D, dtype=torch.bfloat16)
    return bf16(), bf16(), bf16(), torch.ones(*lead), torch.ones(*lead)


@pytest.mark.parametrize("device", ["cpu", "meta"])
def test_tensors_off_the_gpu_are_refused(no_launch, device):
    seq, step = [x.to(device) for x in _args(B, T, H)], [x.to(device) for x in _args(B, H)]
    state = lambda: torch.zeros(B, H, D, D, device=device)
    dy, S = torch.zeros_like(seq[2]), torch.zeros(8, D, device=device)
    for call in (lambda: binding.gka_forward(*seq, 4),
                 lambda: binding.gka_decode_step(state(), state(), *step, 4),
                 lambda: binding.gka_decode_tokens(state(), state(), *seq, 4),
                 lambda: binding.gka_backward(*seq, dy, 4),
                 lambda: binding.gka_backward(*seq, dy, 4, H_init=state(), U_init=state(), return_state_grads=True),
                 lambda: binding.gka_forward_sketched(*seq, S, 4)):
        with pytest.raises(ValueError):
            call()
    assert no_launch == []
