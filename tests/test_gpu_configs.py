"""GPU parity at the full sizes of the five benchmark configurations, through the C ABI, in the launch
configuration bench.py times. The fp64 oracle runs on the host cores on the same seeded inputs."""
import numpy as np
import pytest

import oracle
from paper_2511_21016_amd import binding, synth
from gka_testutil import pair_rel_err, to_device, to_host, upload_inputs

pytestmark = pytest.mark.gpu

TOL_F32 = 1e-4     # max relative error, fp32 configurations
TOL_BF16 = 2e-2    # max relative error, bf16 configurations


def _forward(w, x, compute, **kw):
    import torch
    dev = upload_inputs(x, w.dtype)
    out = binding.gka_forward(dev["q"], dev["k"], dev["v"], dev["gate"], dev["lam"], w.n_iter, compute=compute, **kw)
    torch.cuda.synchronize()
    return out


def test_cfg1_tiny_f32_full():
    w = synth.CFG1
    x = synth.make_inputs(w)
    o = _forward(w, x, binding.GKA_COMPUTE_F32)
    ref = oracle.forward(x["q"], x["k"], x["v"], x["gate"], x["lam"], w.n_iter)
    assert pair_rel_err(to_host(o), ref) <= TOL_F32


def test_cfg2_layer_bf16_full():
    w = synth.CFG2
    x = synth.make_inputs(w)
    o, ex = _forward(w, x, binding.GKA_COMPUTE_BF16, return_fro=True)
    ref, rex = oracle.forward(x["q"], x["k"], x["v"], x["gate"], x["lam"], w.n_iter, return_fro=True)
    err = pair_rel_err(to_host(o), ref)
    print("cfg2 max rel err", err)
    assert err <= TOL_BF16
    assert np.abs(to_host(ex["fro"]) - rex["fro"]).max() <= 5e-3 * rex["fro"].max()


def test_cfg3_long_bf16_full():
    w = synth.CFG3
    x = synth.make_inputs(w)
    o = _forward(w, x, binding.GKA_COMPUTE_BF16)
    y = to_host(o)
    del o
    ref = oracle.forward(x["q"], x["k"], x["v"], x["gate"], x["lam"], w.n_iter)
    err = pair_rel_err(y, ref)
    print("cfg3 max rel err", err)
    assert err <= TOL_BF16


@pytest.mark.parametrize("compute", ["bf16_split", "f32"])
def test_cfg4_illconditioned_full(compute):
    """bf16 tensors, ill-conditioned H_t, at full size: on the bf16 matrix cores with H_[n] and the update as value +
    remainder (GKA_COMPUTE_BF16_SPLIT, the mode for such inputs), and with float32 matrix products."""
    w = synth.CFG4
    x = synth.make_inputs(w)
    o = _forward(w, x, binding.GKA_COMPUTE_BF16_SPLIT if compute == "bf16_split" else binding.GKA_COMPUTE_F32)
    ref = oracle.forward(x["q"], x["k"], x["v"], x["gate"], x["lam"], w.n_iter)
    err = pair_rel_err(to_host(o), ref)
    print("cfg4", compute, "max rel err", err)
    assert err <= TOL_BF16


def test_cfg5_decode_subset():
    """16 of the 256 sequences x 32 heads: prefill 2048 tokens with gka_forward, then 1024 single-token steps with
    gka_decode_step; the oracle follows every step. (Pairs are independent, so a subset of sequences exercises the
    same kernels; the full 256-sequence batch is what the decode benchmark times.)"""
    import torch
    w = synth.CFG5.scaled(B=16)
    n_steps = synth.CFG5_DECODE_STEPS
    x = synth.make_inputs(w)
    o, ex = _forward(w, x, binding.GKA_COMPUTE_F32, return_state=True)
    ref, rex = oracle.forward(x["q"], x["k"], x["v"], x["gate"], x["lam"], w.n_iter, return_state=True)
    assert pair_rel_err(to_host(o), ref) <= TOL_BF16
    Hd, Ud = ex["H_final"], ex["U_final"]
    np.testing.assert_allclose(to_host(Hd), rex["H_final"], rtol=0, atol=2e-5 * np.abs(rex["H_final"]).max())
    np.testing.assert_allclose(to_host(Ud), rex["U_final"], rtol=0, atol=2e-5 * np.abs(rex["U_final"]).max())
    # both sides continue from the GPU's fp32 states
    Hs, Us = to_host(Hd), to_host(Ud)
    steps = synth.make_decode_tokens(w, n_steps)
    dev = {name: to_device(steps[name], w.dtype if name in ("q", "k", "v") else "f32") for name in steps}
    outs = torch.empty((n_steps, w.B, w.H, w.d), dtype=torch.bfloat16, device="cuda")
    for s in range(n_steps):
        binding.gka_decode_step(Hd, Ud, dev["q"][s], dev["k"][s], dev["v"][s], dev["gate"][s], dev["lam"][s],
                                w.n_iter, out=outs[s])
    torch.cuda.synchronize()
    y = to_host(outs)
    worst = 0.0
    for s in range(n_steps):
        r = oracle.decode_step(Hs, Us, steps["q"][s], steps["k"][s], steps["v"][s], steps["gate"][s],
                               steps["lam"][s], w.n_iter)
        e = np.abs(y[s] - r).max(axis=-1) / np.abs(r).max(axis=-1)
        worst = max(worst, float(e.max()))
    print("cfg5 decode max rel err over", n_steps, "steps:", worst)
    assert worst <= TOL_BF16
    np.testing.assert_allclose(to_host(Hd), Hs, rtol=0, atol=1e-4 * np.abs(Hs).max())
    np.testing.assert_allclose(to_host(Ud), Us, rtol=0, atol=1e-4 * np.abs(Us).max())


def test_cfg5_decode_full_batch_sampled():
    """The decode benchmark's launch configuration (256 sequences x 32 heads = 8192 pairs, d = 128): a one-chunk
    prefill with gka_forward, then 8 tokens three ways (single steps on the full H state, single steps on the
    block-lower layout, one gka_decode_tokens call). The oracle follows a seeded sample of 48 pairs from the
    states the prefill left."""
    import torch
    w = synth.CFG5.scaled(T=64)
    n_steps = 8
    x = synth.make_inputs(w)
    o, ex = _forward(w, x, binding.GKA_COMPUTE_F32, return_state=True)
    rng = np.random.default_rng(55)
    flat = rng.choice(w.B * w.H, size=48, replace=False)
    sb, sh = flat // w.H, flat % w.H

    def sample(a):                      # [B,T,H,...] -> [S,T,1,...]
        return np.ascontiguousarray(a[sb, :, sh][:, :, None])

    xs = {name: sample(a) for name, a in x.items()}
    ref, rex = oracle.forward(xs["q"], xs["k"], xs["v"], xs["gate"], xs["lam"], w.n_iter, return_state=True)
    assert pair_rel_err(sample(to_host(o)), ref) <= TOL_BF16
    Hd, Ud = ex["H_final"], ex["U_final"]
    Hs = np.ascontiguousarray(to_host(Hd)[sb, sh][:, None])          # the oracle continues from the GPU's fp32 states
    Us = np.ascontiguousarray(to_host(Ud)[sb, sh][:, None])
    steps = synth.make_decode_tokens(w, n_steps)                     # [n_steps, B, H, ...]
    dev = {name: to_device(steps[name], w.dtype if name in ("q", "k", "v") else "f32") for name in steps}
    H_full, U_full = Hd.clone(), Ud.clone()
    H_low, U_low = Hd.clone(), Ud.clone()
    H_multi, U_multi = Hd.clone(), Ud.clone()
    out_full = torch.empty((n_steps, w.B, w.H, w.d), dtype=torch.bfloat16, device="cuda")
    out_low = torch.empty_like(out_full)
    for s in range(n_steps):
        binding.gka_decode_step(H_full, U_full, dev["q"][s], dev["k"][s], dev["v"][s], dev["gate"][s], dev["lam"][s],
                                w.n_iter, out=out_full[s])
        binding.gka_decode_step(H_low, U_low, dev["q"][s], dev["k"][s], dev["v"][s], dev["gate"][s], dev["lam"][s],
                                w.n_iter, out=out_low[s], state_layout=binding.GKA_STATE_H_LOWER_BLOCKS)
    bt = {name: dev[name].transpose(0, 1).contiguous() for name in dev}          # [B, n_steps, H, ...]
    out_multi = binding.gka_decode_tokens(H_multi, U_multi, bt["q"], bt["k"], bt["v"], bt["gate"], bt["lam"], w.n_iter)
    torch.cuda.synchronize()
    ys = {"full": to_host(out_full)[:, sb, sh], "lower": to_host(out_low)[:, sb, sh],
          "multi": np.moveaxis(to_host(out_multi)[sb, :, sh], 0, 1)}            # [n_steps, S, d]
    worst = dict.fromkeys(ys, 0.0)
    for s in range(n_steps):
        r = oracle.decode_step(Hs, Us, *(np.ascontiguousarray(steps[n][s][sb, sh][:, None])
                                         for n in ("q", "k", "v", "gate", "lam")), w.n_iter)[:, 0]
        for name, y in ys.items():
            e = np.abs(y[s] - r).max(axis=-1) / np.abs(r).max(axis=-1)
            worst[name] = max(worst[name], float(e.max()))
    print("cfg5 full batch, sampled pairs, max rel err:", worst)
    assert max(worst.values()) <= TOL_BF16
    assert torch.equal(out_full, out_multi.transpose(0, 1))          # the same kernel arithmetic token by token
    for Hx, Ux in ((H_full, U_full), (H_low, U_low), (H_multi, U_multi)):
        hh = to_host(Hx)[sb, sh][:, None]
        if Hx is H_low:                                              # only the block-lower part is maintained
            i, j = np.meshgrid(np.arange(w.d), np.arange(w.d), indexing="ij")
            keep = j < 32 * (i // 32 + 1)
            hh = np.where(keep, hh, Hs)
        np.testing.assert_allclose(hh, Hs, rtol=0, atol=1e-4 * np.abs(Hs).max())
        np.testing.assert_allclose(to_host(Ux)[sb, sh][:, None], Us, rtol=0, atol=1e-4 * np.abs(Us).max())


def test_cfg2_backward_and_sketch_full_size_sampled():
    """The backward pass and the sketched forward at the size and in the launch configuration that bench.py times
    (64 pairs x 4096 tokens: 4 scan segments in the solves, 8 in the plain readouts), checked on three sampled
    (batch, head) pairs that the numpy oracles can follow one by one."""
    import torch
    from oracle import gka_backward_oracle as bwd
    from oracle import gka_sketch_oracle as sk
    w = synth.CFG2
    x = synth.make_inputs(w)
    rng = np.random.default_rng(99)
    dy = synth.round_to_bf16(rng.standard_normal(x["v"].shape).astype(np.float32))
    dev = upload_inputs(x, w.dtype)
    out = binding.gka_backward(dev["q"], dev["k"], dev["v"], dev["gate"], dev["lam"], to_device(dy, "bf16"), w.n_iter)
    S = (rng.standard_normal((w.H, 32, w.d)) / np.sqrt(w.d)).astype(np.float32)
    ys = binding.gka_forward_sketched(dev["q"], dev["k"], dev["v"], dev["gate"], dev["lam"], to_device(S, "f32"),
                                      w.n_iter)
    torch.cuda.synchronize()
    got = {n: to_host(out[n]) for n in ("dq", "dk", "dv", "dgate", "dlam")}
    ys = to_host(ys)
    for b, h in ((0, 0), (2, 7), (3, 15)):
        sel = lambda a: a[b, :, h]
        ref = bwd.backward_pair(sel(x["q"]), sel(x["k"]), sel(x["v"]), sel(x["gate"]), sel(x["lam"]), sel(dy),
                                w.n_iter)
        errs = {n: float(np.abs(sel(got[n]) - ref[n]).max() / np.abs(ref[n]).max()) for n in got}
        print("cfg2 backward pair", b, h, errs)
        # bf16 tensors, the stated tolerance for every gradient (measured: dk 1.3-1.5 %, the gate gradient, a
        # cumulative sum over the rest of the sequence, 0.2-1.1 %, the rest below 0.7 %)
        assert max(errs.values()) <= TOL_BF16, errs
        yref = sk.forward_sketched_pair(sel(x["q"]), sel(x["k"]), sel(x["v"]), sel(x["gate"]), sel(x["lam"]), S[h],
                                        w.n_iter)
        es = float(np.abs(sel(ys) - yref).max() / np.abs(yref).max())
        print("cfg2 sketched pair", b, h, es)
        assert es <= TOL_BF16, es


@pytest.mark.parametrize("compute", ["bf16", "f32"])
def test_cfg3_shape_backward_long_sequence(compute):
    """A long sequence (configuration 3's shape with two heads: T = 32768, 512 chunks per pair, 256 scan segments in
    the readouts) against the backward oracle on one pair (the oracle keeps every state of that pair: 8.6 GB, 10 s).
    The gate gradient is a cumulative sum over up to 32768 tokens: it stays near 2 % because the pieces of the sum
    are formed from the stored tensors with value + remainder operands and handed over in float32."""
    import torch
    from oracle import gka_backward_oracle as bwd
    w = synth.CFG3.scaled(H=2, seed=31)
    x = synth.make_inputs(w)
    rng = np.random.default_rng(5)
    dy = synth.round_to_bf16(rng.standard_normal(x["v"].shape).astype(np.float32))
    dev = upload_inputs(x, w.dtype)
    cm = binding.GKA_COMPUTE_BF16 if compute == "bf16" else binding.GKA_COMPUTE_F32
    out = binding.gka_backward(dev["q"], dev["k"], dev["v"], dev["gate"], dev["lam"], to_device(dy, "bf16"), w.n_iter,
                               compute=cm)
    torch.cuda.synchronize()
    sel = lambda a: a[0, :, 1]
    ref = bwd.backward_pair(sel(x["q"]), sel(x["k"]), sel(x["v"]), sel(x["gate"]), sel(x["lam"]), sel(dy), w.n_iter)
    errs = {n: float(np.abs(sel(to_host(out[n])) - ref[n]).max() / np.abs(ref[n]).max())
            for n in ("dq", "dk", "dv", "dgate", "dlam")}
    print("cfg3-shape backward,", compute, "operands:", errs)
    # the stated bf16 tolerance, but for the gate gradient: a cumulative sum over up to 32768 tokens of differences
    # of products; measured 1.9 % with bf16 and with float32 operands, the rest below 1.3 %
    assert max(errs[n] for n in ("dq", "dk", "dv", "dlam")) <= TOL_BF16, errs
    assert errs["dgate"] <= 3e-2, errs
