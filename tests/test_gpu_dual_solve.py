"""Both solves of the backward pass in the fused kernels' walk (bf16 tensors, d = 128): against the oracle around the edges of
chunks and chunk pairs, with every option, in segments and from initial states; gradients that replace their inputs."""
import numpy as np
import pytest

from oracle import gka_backward_oracle as bwd
from paper_2511_21016_amd import binding, synth
from gka_testutil import to_device, to_host, upload_inputs

pytestmark = pytest.mark.gpu

# Bounds of test_gpu_backward.py, of a gradient's largest value: 2e-2 against the oracle, 5e-2 for dk of short sequences under
# the rule, 3e-2 for dalpha of a single token. Between two paths that both meet them: twice that. Some of the random systems here
# are conditioned so badly (lambda of 0.01, 8 passes) that the rounding of their bf16 operands alone exceeds these bounds; there the
# error of the two-phase solve, which rounds the same operands, was measured before the walk was there, and a quarter more is
# allowed: the sums and the start states are not formed in the same order. (T, variants, rule): {gradient: that error}
TOL, TOL_DK_RULE, TOL_DALPHA_ONE = 2e-2, 5e-2, 3e-2
ILL_CONDITIONED = {(1, False, 0.0): {"dk": 0.0299}, (1, True, 0.0): {"dk": 0.0322, "dalpha": 0.1388},
                   (1, True, 0.05): {"dk": 0.0859, "dv": 0.0316, "dalpha": 0.1869}, (129, False, 0.0): {"dk": 0.0206},
                   (200, False, 0.0): {"dlam": 0.0416}}


def run(w, x, dy, path, walk_chunks=0, variants=False, rule=0.0, in_place=False, states=None):
    import torch
    B, T, H, d = x["q"].shape
    dev = upload_inputs(x, "bf16")
    dyd = to_device(dy, "bf16")
    lam = None if rule else dev["lam"]
    beta = alpha = None
    if variants:
        g = synth.make_gates(w)
        beta, alpha = to_device(g["beta"], "f32"), to_device(g["alpha"], "f32")
    ptr = lambda t: None if t is None else t.data_ptr()
    p = binding.make_params(B, H, T, d, w.n_iter, binding.GKA_BF16, binding.GKA_COMPUTE_BF16, lambda_scale=rule, beta=ptr(beta),
                            alpha=ptr(alpha), path=path, walk_chunks=walk_chunks)
    nbytes = binding.backward_workspace_bytes(p)
    ws = torch.full((nbytes // 4 + 64,), float("nan"), device="cuda")
    out = {n: torch.empty((B, T, H, d), device="cuda") for n in ("dq", "dk", "dv")}
    out["dgate"] = torch.empty((B, T, H), device="cuda")
    for n, src in (("dlam", lam), ("dbeta", beta), ("dalpha", alpha)):
        if src is not None:
            out[n] = src if in_place else torch.empty_like(src)
    Hi, Ui = states or (None, None)
    st = binding.backward_from_state_raw(p, ptr(dev["q"]), ptr(dev["k"]), ptr(dev["v"]), ptr(dev["gate"]), ptr(lam), ptr(dyd),
                                         ptr(Hi), ptr(Ui), ptr(out["dq"]), ptr(out["dk"]), ptr(out["dv"]), ptr(out["dgate"]),
                                         ptr(out.get("dlam")), ptr(out.get("dbeta")), ptr(out.get("dalpha")),
                                         workspace=ptr(ws), workspace_bytes=nbytes, stream=torch.cuda.current_stream().cuda_stream)
    assert st == binding.GKA_OK, binding.status_string(st)
    torch.cuda.synchronize()
    return {n: to_host(t) for n, t in out.items()}


def problem(B, H, T, n_iter=8, seed=0):
    w = synth.CFG2.scaled(B=B, H=H, T=T, d=128, n_iter=n_iter, seed=6100 + T + seed)
    x = synth.make_inputs(w)
    dy = synth.round_to_bf16(np.random.default_rng(w.seed).standard_normal(x["v"].shape).astype(np.float32))
    return w, x, dy


def compare(got, want, T, rule, factor=1, known={}):
    for n in got:
        if n == "dgate" and T == 1:          # the gate multiplies a zero state: what is left of terms of order one
            assert np.abs(got[n]).max() <= 2e-3
            continue
        tol = TOL_DK_RULE if n == "dk" and rule else TOL_DALPHA_ONE if n == "dalpha" and T == 1 else TOL
        tol *= factor
        err = np.abs(got[n] - want[n]).max() / np.abs(want[n]).max()
        if n in known:
            tol = 1.25 * known[n]
        assert np.isfinite(got[n]).all() and err <= tol, (n, err, tol)


@pytest.mark.parametrize("T", [1, 16, 63, 64, 65, 127, 128, 129, 200, 390])
@pytest.mark.parametrize("variants,rule", [(False, 0.0), (True, 0.0), (True, 0.05)])
def test_against_the_oracle(T, variants, rule):
    w, x, dy = problem(2, 3, T)
    print("dual solve", T, variants, rule, flush=True)
    got = run(w, x, dy, binding.GKA_PATH_AUTO, variants=variants, rule=rule)
    opt = synth.make_gates(w) if variants else {}
    want = bwd.backward(x["q"], x["k"], x["v"], x["gate"], None if rule else x["lam"], dy, w.n_iter, lambda_scale=rule,
                        **{n: opt[n] for n in ("beta", "alpha") if n in opt})
    compare(got, want, T, rule, known=ILL_CONDITIONED.get((T, variants, rule), {}))


@pytest.mark.parametrize("walk", [2, 4, 6])
def test_segments_initial_states_and_wiped_states(walk):
    import torch
    w, x, dy = problem(1, 3, 700, seed=walk)
    x["gate"][0, 100, 1] = 0.0               # a packed sequence begins inside a chunk,
    x["gate"][0, 128, 2] = 0.0               # at the beginning of one
    gen = torch.Generator(device="cuda").manual_seed(walk)
    A = torch.randn((1, 3, 128, 8), generator=gen, device="cuda")
    Hi = torch.matmul(A, A.transpose(-1, -2).contiguous()) / 8
    Hi = 0.5 * (Hi + Hi.transpose(-1, -2).contiguous())
    Ui = 0.1 * torch.randn((1, 3, 128, 128), generator=gen, device="cuda")
    for states in (None, (Hi, Ui)):
        got = run(w, x, dy, binding.GKA_PATH_AUTO, walk_chunks=walk, states=states)
        compare(got, run(w, x, dy, binding.GKA_PATH_TWO_PHASE, states=states), 700, 0.0, factor=2)
        H, U = (s.cpu().numpy() for s in states) if states else (None, None)
        want = bwd.backward(x["q"], x["k"], x["v"], x["gate"], x["lam"], dy, w.n_iter, H_init=H, U_init=U)
        want["dgate"][x["gate"] == 0.0] = 0.0                # (reported as 0 at a gate of 0)
        compare(got, want, 700, 0.0)


@pytest.mark.parametrize("n_iter", [0, 1])
def test_few_passes(n_iter):
    w, x, dy = problem(1, 2, 150, n_iter=n_iter)
    compare(run(w, x, dy, binding.GKA_PATH_AUTO), run(w, x, dy, binding.GKA_PATH_TWO_PHASE), 150, 0.0, factor=2)


def test_gradients_of_scalars_over_their_inputs():
    """dlambda, dbeta and dalpha in the buffers of lambda, beta and alpha: the same bits as in buffers of their own."""
    w, x, dy = problem(2, 2, 300)
    got = run(w, x, dy, binding.GKA_PATH_AUTO, variants=True, in_place=True)
    want = run(w, x, dy, binding.GKA_PATH_AUTO, variants=True)
    for n in want:
        assert (got[n] == want[n]).all(), n


@pytest.mark.parametrize("T", [200, 390])
def test_operands_are_rounded_as_the_two_phase_solve_rounds_them(T):
    """The error is that of the bf16 operands. With the same operands on both paths most of it is common to them: they are nearer
    to each other than half the error. Other roundings (of a system divided by zeta_c, say) would leave independent errors of
    the same size, 1.4 times it apart."""
    w, x, dy = problem(2, 3, T, seed=50)
    got = run(w, x, dy, binding.GKA_PATH_AUTO)
    other = run(w, x, dy, binding.GKA_PATH_TWO_PHASE)
    want = bwd.backward(x["q"], x["k"], x["v"], x["gate"], x["lam"], dy, w.n_iter)
    for n in ("dq", "dk", "dv", "dlam"):
        ref = np.asarray(want[n], dtype=np.float64)
        apart, err = np.linalg.norm(got[n] - other[n]), np.linalg.norm(other[n] - ref)
        print(T, n, apart / err, flush=True)
        assert apart <= 0.5 * err, (n, apart / err)
    # The gate gradient is a cumulative sum in which almost everything cancels: what is left follows the order of the sums and of the
    # start states, so that the two errors are of one size but independent, 1.4 times it apart (half as much again for six pairs)
    ref = np.asarray(want["dgate"], dtype=np.float64)
    errs = [np.linalg.norm(a["dgate"] - ref) for a in (got, other)]
    print(T, "dgate", errs[0] / errs[1], flush=True)
    assert np.linalg.norm(got["dgate"] - other["dgate"]) <= 2.1 * errs[1] and errs[0] <= 2.0 * errs[1]


def test_more_pairs_than_workgroups_in_four_rounds():
    """1088 pairs of three chunks: each pair's gradients are those of a call with fewer pairs and the same segments, bit for bit,
    and the pass keeps within a workspace of the size that the query gives."""
    import torch
    B, H, T = 64, 17, 150
    w = synth.CFG2.scaled(B=2, H=H, T=T, d=128, n_iter=4, seed=6400)
    x = synth.make_inputs(w)
    dy = synth.round_to_bf16(np.random.default_rng(w.seed).standard_normal(x["v"].shape).astype(np.float32))
    dev = upload_inputs(x, "bf16")
    few = [dev[n] for n in ("q", "k", "v", "gate", "lam")] + [to_device(dy, "bf16")]
    many = [t.repeat(B // 2, *[1] * (t.dim() - 1)).contiguous() for t in few]
    p = binding.make_params(B, H, T, 128, w.n_iter, binding.GKA_BF16, binding.GKA_COMPUTE_BF16)
    nbytes = binding.backward_workspace_bytes(p)
    ws = torch.full((nbytes + (64 << 20),), 255, dtype=torch.uint8, device="cuda")
    ws[nbytes:] = 77
    print("backward pass of", B * H, "pairs", flush=True)
    got = binding.gka_backward(*many, w.n_iter, workspace=ws[:nbytes])
    torch.cuda.synchronize()
    assert bool((ws[nbytes:] == 77).all())
    want = run(w, x, dy, binding.GKA_PATH_AUTO, walk_chunks=3)
    for n, a in got.items():
        a = to_host(a)
        assert all((a[i:i + 2] == want[n]).all() for i in range(0, B, 2)), n
    x1 = {n: a[:1, :, :2] for n, a in x.items()}
    ref = bwd.backward(x1["q"], x1["k"], x1["v"], x1["gate"], x1["lam"], dy[:1, :, :2], w.n_iter)
    compare({n: a[:1, :, :2] for n, a in want.items()}, ref, T, 0.0)


def test_lambda_gradient_takes_x_in_float32():
    """Without passes x_t = 2 q_t / (L + mu), p_t is dq_t, and dlambda_t = -x_t . p_t can be formed from them: 128 float32
    products and sums, a relative 2^-24 for each rounding of a partial sum and for the common factor. x as bf16 value +
    remainder, 2^-18 of every element, would leave three to five times as much."""
    w, x, dy = problem(2, 4, 300, n_iter=0, seed=90)
    x["lam"] = (x["lam"] + 1024.0).astype(np.float32)
    got = run(w, x, dy, binding.GKA_PATH_AUTO)
    dev = upload_inputs(x, "bf16")
    fro = to_host(binding.gka_forward(*(dev[n] for n in ("q", "k", "v", "gate", "lam")), 0, return_fro=True)[1]["fro"])
    terms = 2.0 * x["q"].astype(np.float64) / (fro + 2.0 * x["lam"])[..., None] * got["dq"]
    err = np.abs(got["dlam"] + terms.sum(axis=-1)) / np.abs(terms).sum(axis=-1)
    print("dlambda", err.max(), np.sqrt((err ** 2).mean()), flush=True)
    assert err.max() <= 2e-7
