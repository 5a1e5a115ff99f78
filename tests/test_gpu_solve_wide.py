"""d = 256, bf16 tensors: the solve on 16-bit pieces against the kernel with float32 products, which float32 tensors of the same
values run on. Both have float32's precision: they differ by its roundings, which systems of condition number up to about 2000
(lambda down to 1e-2) amplify."""
import numpy as np
import pytest

from paper_2511_21016_amd import binding, synth
from gka_testutil import to_device, to_host

pytestmark = pytest.mark.gpu

# 2^-24 per rounding, about 2^4 of them in a row of 256 products and 2000 from the condition number: 2e-3 is the worst case, a
# hundredth of it what random signs leave (measured: 1e-5)
TOL = 2e-5


def both(x, n_iter, variants=None, of=("bf16", "f32"), compute=None, **kw):
    import torch
    out = []
    for dtype in of:
        dev = {n: to_device(x[n], dtype) for n in ("q", "k", "v")}
        opt = {n: to_device(v, "f32") for n, v in (variants or {}).items()}
        o, ex = binding.gka_forward(dev["q"], dev["k"], dev["v"], to_device(x["gate"], "f32"),
                                    None if "lambda_scale" in kw else to_device(x["lam"], "f32"), n_iter, return_xhat=True,
                                    return_fro=True, return_state=True, compute=compute, **opt, **kw)
        torch.cuda.synchronize()
        out.append({"o": to_host(o), **{n: to_host(t) for n, t in ex.items()}})
    return out


def check(got, want, tol=TOL):
    for n in ("xhat", "fro", "H_final", "U_final"):
        scale = np.abs(want[n]).max(axis=(-1, -2) if n.endswith("final") else -1 if n == "xhat" else (1,), keepdims=True)
        assert np.isfinite(got[n]).all(), n
        err = (np.abs(got[n] - want[n]) / np.maximum(scale, 1e-300)).max()
        assert err <= tol, (n, err)
    # the output's own rounding to bf16
    pair = np.abs(want["o"]).max(axis=(1, 3), keepdims=True)
    assert (np.abs(got["o"] - want["o"]) / pair).max() <= 2.0 ** -8


@pytest.mark.parametrize("B,H,T", [(1, 2, 129), (1, 2, 175), (1, 3, 192), (2, 3, 300), (5, 8, 200), (4, 8, 449)])
@pytest.mark.parametrize("variants", [False, True])
def test_against_float32_products(B, H, T, variants):
    w = synth.CFG2.scaled(B=B, H=H, T=T, d=256, n_iter=8, seed=900 + T)
    x = synth.make_inputs(w)
    print("wide", B, H, T, variants, flush=True)
    if variants:
        g = synth.make_gates(w)
        g["beta"][0, 70] = 0.0
        check(*both(x, 8, variants={n: g[n] for n in ("beta", "alpha")}, lambda_scale=0.05))
    else:
        check(*both(x, 8))


@pytest.mark.parametrize("B,H,T", [(1, 2, 175), (4, 8, 300)])
def test_float32_operands_of_bf16_tensors(B, H, T):
    """GKA_COMPUTE_F32 is the float32 MFMA path for either type of tensors: the same bits up to the output's rounding."""
    w = synth.CFG2.scaled(B=B, H=H, T=T, d=256, n_iter=8, seed=950 + T)
    x = synth.make_inputs(w)
    got, want = both(x, 8, compute=binding.GKA_COMPUTE_F32)
    for n in ("xhat", "fro", "H_final", "U_final"):
        assert (got[n] == want[n]).all(), n
    assert (got["o"] == synth.round_to_bf16(want["o"].astype(np.float32))).all()


@pytest.mark.parametrize("n_iter", [0, 1, 60, 61])
def test_numbers_of_passes(n_iter):
    """60 passes are the last on this kernel (the updates' scale leaves room for their growth up to there)."""
    w = synth.CFG2.scaled(B=1, H=2, T=140, d=256, n_iter=n_iter, seed=77)
    check(*both(synth.make_inputs(w), n_iter))


@pytest.mark.parametrize("scale_q,scale_k,scale_v", [(2.0 ** -70, 1.0, 1.0), (2.0 ** 60, 2.0 ** 5, 2.0 ** 40), (1.0, 2.0 ** -12, 2.0 ** -60)])
def test_scales(scale_q, scale_k, scale_v):
    """Powers of two far from one in q, k and v, with lambda scaled like the states: the same numbers up to that scale, so that a
    scale chosen wrongly shows as lost digits. Single tokens are zero, single keys a thousand times smaller."""
    w = synth.CFG2.scaled(B=1, H=2, T=200, d=256, n_iter=8, seed=78)
    x = synth.make_inputs(w)
    x["q"][0, 5] = 0.0
    x["k"][0, 9] = 0.0
    x["k"][0, 100:110] *= 2.0 ** -10
    for n, s in (("q", scale_q), ("k", scale_k), ("v", scale_v)):
        x[n] = (x[n] * s).astype(np.float32)
    x["lam"] = (x["lam"] * scale_k ** 2).astype(np.float32)
    check(*both(x, 8))


def test_features_of_other_scales():
    """Single features of q, k and v are 2^-32 of the others: their rows of the states are as small, and what the solve and the
    readout make of them has float32's and the output's precision by itself."""
    w = synth.CFG2.scaled(B=1, H=2, T=200, d=256, n_iter=8, seed=80)
    x = synth.make_inputs(w)
    few = [5, 40, 200]
    for n in ("q", "k", "v"):
        x[n][..., few] *= np.float32(2.0 ** -32)
    got, want = both(x, 8)
    check(got, want)
    for n, tol in (("xhat", TOL), ("o", 2.0 ** -8)):
        scale = np.abs(want[n][..., few]).max(axis=1, keepdims=True)
        assert (np.abs(got[n][..., few] - want[n][..., few]) / scale).max() <= tol, n


def test_small_elements_of_keys():
    """Queries live where every key is 2^-22 of its largest element: the products of keys and vectors are sums of those small
    elements, which count with all their bits. (Lambda is so large that the solve does not turn the vectors to the others, where
    elements 2^-28 of the largest would count.)"""
    w = synth.CFG2.scaled(B=1, H=2, T=200, d=256, n_iter=8, seed=81)
    x = synth.make_inputs(w)
    x["q"][..., :128] = 0.0
    x["k"][..., 128:] *= np.float32(2.0 ** -22)
    x["lam"] += np.float32(4096.0)
    check(*both(x, 8))


def test_a_wiped_state_and_a_tiny_key_behind_it():
    w = synth.CFG2.scaled(B=1, H=2, T=200, d=256, n_iter=8, seed=79)
    x = synth.make_inputs(w)
    x["gate"][0, 100] = 0.0
    x["k"][0, 100:] *= 2.0 ** -13
    x["lam"][0, 100:] *= 2.0 ** -26
    check(*both(x, 8), tol=1e-4)          # (what exp(-100) leaves of the old state is not negligible beside 2^-26 in the same way)


@pytest.mark.parametrize("T,n_iter", [(150, 20), (200, 30), (129, 60)])
@pytest.mark.parametrize("variants", [False, True])
def test_initial_states_that_are_not_positive_semidefinite(T, n_iter, variants):
    """Eigenvalues below zero lie outside the interval that the iteration is made for and its updates grow, thousandfold in ten
    passes: they are scaled down on the way, and what comes out is what float32 products give. A pass's products are right to
    2^-22 of their operands' size on either side; where everything grows these errors add up, n_iter of them (a factor of four
    for their number and for elements that are larger than the common size). Behind a wiped state in the same chunk nothing grows."""
    w = synth.CFG2.scaled(B=1, H=2, T=T, d=256, n_iter=n_iter, seed=82)
    x = synth.make_inputs(w)
    x["gate"][:] = 1.0 - 2.0 ** -12                  # (the initial state stays,
    x["gate"][0, 100, 1] = 0.0                       # but for the second pair's)
    A = np.random.default_rng(82).standard_normal((1, 2, 256, 256)).astype(np.float32)
    kw = dict(H_init=to_device(A + A.transpose(0, 1, 3, 2), "f32"), U_init=to_device(A, "f32"))
    if variants:
        g = synth.make_gates(w)
        kw["variants"] = {n: g[n] for n in ("beta", "alpha")}
    print("not semidefinite", T, n_iter, variants, flush=True)
    got, want = both(x, n_iter, **kw)
    first = np.abs(2.0 * x["q"] / (want["fro"] + 2.0 * x["lam"])[..., None])
    for pair, tokens in ((0, slice(0, T)), (1, slice(0, 100)), (1, slice(100, 128))):
        a, b = (y["xhat"][0, tokens, pair] for y in (got, want))
        grown, err = np.abs(b).max() / first[0, tokens, pair].max(), np.abs(a - b).max() / np.abs(b).max()
        print(pair, tokens, grown, err, flush=True)
        assert np.isfinite(b).all() and (grown > 2.0 ** 14) == (tokens.start == 0)
        assert np.isfinite(got["o"]).all() and err <= n_iter * 2.0 ** -20
