"""The work that programs have libgka do, as a list of measurable cases.

A case is one call of a public entry point of `paper_2511_21016_amd.binding` on tensors that live in HBM, the way a
serving loop or a training step makes it: workspace and output buffers are kept by the caller, nothing synchronises.
Inputs follow the distributions of the synthetic workloads of this package (`synth.py`), drawn on the device:
L2-normalised q and k, v ~ N(0, 1), gates sigmoid(N(m, 1)), lambda = softplus(N(0, 1)) + 1e-2.

Kinds of case
  decode     one recurrent token per (sequence, head) on stored float32 states, in place
  tokens     a few tokens per call on stored states (speculative or multi-token decoding)
  forward    whole sequences: prefill, the forward half of training, long contexts, ill-conditioned systems
  backward   the gradients of a whole sequence
  sketched   the forward pass with latent sketching
"""
import math

import torch

from paper_2511_21016_amd import binding

_DTYPES = {"bf16": torch.bfloat16, "f32": torch.float32}
_COMPUTE = {"default": None, "split": binding.GKA_COMPUTE_BF16_SPLIT}

# Values that a case leaves out.
_DEFAULTS = {
    "dtype": "bf16",        # of q, k, v, o
    "r": 10,                # Chebyshev passes
    "rule": False,          # lambda_t = 0.02 ||H_t||_F, else lambda is given per token
    "beta": False,          # write gate
    "alpha": False,         # alpha-connection
    "states": False,        # forward: the final states are asked for (prefill)
    "lower": False,         # decode cache that keeps the block-lower triangle of H
    "compute": "default",   # "split": bf16 value + remainder operands
    "rank": 0,              # > 0: keys from a subspace of this rank (ill-conditioned systems)
    "gate_mean": 3.0,
    "d_s": 0,               # sketch dimension
}
_RULE_SCALE = 0.02


def listed():
    return [
        # --- decoding
        # one interactive sequence: the smallest call, where launch and latency count
        {"name": "decode_1_sequence", "kind": "decode", "B": 1, "H": 16, "T": 1, "d": 128},
        # a full serving batch: 256 sequences of a 32-head layer
        {"name": "decode_256_sequences", "kind": "decode", "B": 256, "H": 32, "T": 1, "d": 128},
        # speculative decoding: four tokens per call for 48 sequences, the compact cache of H
        {"name": "decode_4_tokens", "kind": "tokens", "B": 48, "H": 32, "T": 4, "d": 128, "lower": True},
        # --- whole sequences
        # one prompt of an ordinary, odd length with the layer's own rule for lambda, its write gate and
        # alpha-connection; the states go to the decode cache
        {"name": "prefill_prompt", "kind": "forward", "B": 1, "H": 16, "T": 1337, "d": 128, "rule": True, "beta": True,
         "alpha": True, "states": True},
        # the forward half of a training step of a 4K-context layer
        {"name": "forward_4k", "kind": "forward", "B": 4, "H": 16, "T": 4096, "d": 128},
        # long context: 32K tokens, 32 heads
        {"name": "forward_32k", "kind": "forward", "B": 1, "H": 32, "T": 32768, "d": 128, "gate_mean": 4.0},
        # ill-conditioned systems (keys of rank 16, small lambda), more passes, value + remainder operands
        {"name": "forward_ill_conditioned", "kind": "forward", "B": 2, "H": 8, "T": 8192, "d": 128, "r": 16, "rank": 16,
         "compute": "split"},
        # float32 tensors at a small size: numerics work, unit-test-like calls
        {"name": "forward_f32_small", "kind": "forward", "B": 1, "H": 1, "T": 256, "d": 64, "dtype": "f32", "r": 8,
         "gate_mean": 2.0},
        # a vision model's layer: many short sequences of 197 tokens, head dimension 16
        {"name": "forward_vision_d16", "kind": "forward", "B": 256, "H": 24, "T": 197, "d": 16},
        # wide heads
        {"name": "forward_d256", "kind": "forward", "B": 4, "H": 8, "T": 1024, "d": 256},
        # latent sketching of the 4K-context layer in 32 dimensions
        {"name": "sketched_4k", "kind": "sketched", "B": 4, "H": 16, "T": 4096, "d": 128, "d_s": 32},
        # --- training: the gradients of the 4K-context layer
        {"name": "backward_4k", "kind": "backward", "B": 4, "H": 16, "T": 4096, "d": 128},
    ]


def _log_int(rng, lo, hi):
    """An integer spread over the logarithm of [lo, hi]."""
    return max(lo, min(hi, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


def _tokens(rng, lo, hi, pairs, budget):
    """A sequence length in [lo, hi], odd ones among them, with pairs * T <= budget."""
    t = _log_int(rng, lo, max(lo, min(hi, budget // pairs)))
    return t if rng.random() < 0.6 or t < 64 else max(lo, t // 64 * 64)


def _variant(rng, case):
    """The layer's options, each in use now and then."""
    for name in ("rule", "beta", "alpha"):
        if rng.random() < 0.3:
            case[name] = True
    return case


def draw(rng):
    kind = rng.choice(("decode", "decode", "tokens", "forward", "forward", "forward", "split", "f32", "small", "wide",
                       "sketched", "backward", "backward"))
    if kind in ("decode", "tokens"):
        H = rng.choice((4, 8, 12, 16, 24, 32))
        case = {"kind": kind, "B": _log_int(rng, 1, 256 if kind == "decode" else 96), "H": H,
                "T": 1 if kind == "decode" else rng.randint(2, 8), "d": rng.choice((128, 128, 64))}
        case["lower"] = rng.random() < 0.4
        case["r"] = rng.choice((8, 10, 10, 12))
        return _variant(rng, case)
    if kind == "forward":
        B, H = _log_int(rng, 1, 16), rng.choice((4, 8, 12, 16, 24, 32))
        case = {"kind": kind, "B": B, "H": H, "T": _tokens(rng, 48, 32768, B * H, 1 << 20), "d": rng.choice((128, 128, 64))}
        case["states"] = rng.random() < 0.5
        case["r"] = rng.choice((8, 10, 10, 12))
        return _variant(rng, case)
    if kind == "split":
        B, H = rng.randint(1, 4), rng.choice((4, 8, 12, 16))
        return {"kind": "forward", "B": B, "H": H, "T": _tokens(rng, 200, 8192, B * H, 1 << 17), "d": 128,
                "r": rng.choice((12, 16)), "rank": 16, "compute": "split"}
    if kind == "f32":
        B, H = rng.randint(1, 4), rng.choice((1, 2, 4, 8, 16))
        return {"kind": "forward", "B": B, "H": H, "T": _tokens(rng, 40, 4096, B * H, 1 << 16), "d": rng.choice((64, 128)),
                "dtype": "f32", "r": rng.choice((8, 10)), "gate_mean": 2.0}
    if kind == "small":
        B, H = _log_int(rng, 8, 256), rng.choice((3, 6, 12, 24))
        return _variant(rng, {"kind": "forward", "B": B, "H": H, "T": _tokens(rng, 50, 785, B * H, 1 << 20),
                              "d": rng.choice((16, 16, 32))})
    if kind == "wide":
        B, H = rng.randint(1, 8), rng.choice((4, 8))
        return {"kind": "forward", "B": B, "H": H, "T": _tokens(rng, 64, 1024, B * H, 1 << 15), "d": 256,
                "states": rng.random() < 0.5}
    if kind == "sketched":
        B, H = rng.randint(1, 8), rng.choice((8, 12, 16, 32))
        return {"kind": kind, "B": B, "H": H, "T": _tokens(rng, 200, 8192, B * H, 1 << 18), "d": 128,
                "d_s": rng.choice((8, 16, 24, 32, 32, 48, 64))}
    B, H = rng.randint(1, 8), rng.choice((4, 8, 12, 16))
    return _variant(rng, {"kind": "backward", "B": B, "H": H, "T": _tokens(rng, 100, 8192, B * H, 1 << 18),
                          "d": rng.choice((128, 128, 64)), "r": rng.choice((8, 10, 10))})


def _full(case):
    return {**_DEFAULTS, **case}


def prepare(case, seed):
    c = _full(case)
    gen = torch.Generator(device="cuda").manual_seed(int(seed))
    B, H, T, d, dt = c["B"], c["H"], c["T"], c["d"], _DTYPES[c["dtype"]]
    f32 = dict(device="cuda", dtype=torch.float32)

    def normal(*shape):
        return torch.randn(shape, generator=gen, **f32)

    def rows(*shape):
        return torch.nn.functional.normalize(normal(*shape), dim=-1)

    def keys(*shape):
        if not c["rank"]:
            return rows(*shape)
        basis = normal(shape[0], 1, shape[2], c["rank"], d)
        coeff = normal(*shape[:-1], c["rank"])
        k = 1e-3 * normal(*shape)
        for i in range(c["rank"]):
            k += coeff[..., i:i + 1] * basis[:, :, :, i]
        return torch.nn.functional.normalize(k, dim=-1)

    lead = (B, H) if c["kind"] == "decode" else (B, T, H)
    s = {"case": c, "q": rows(*lead, d).to(dt), "k": keys(*lead, d).to(dt), "v": normal(*lead, d).to(dt),
         "gate": torch.sigmoid(normal(*lead) + c["gate_mean"]), "lam": None, "beta": None, "alpha": None}
    if not c["rule"]:
        scale, offset = (1e-3, 0.0) if c["rank"] else (1.0, 1e-2)
        s["lam"] = scale * torch.nn.functional.softplus(normal(*lead)) + offset
    for name in ("beta", "alpha"):
        if c[name]:
            s[name] = torch.sigmoid(normal(*lead) + 1.0)
    s["lambda_scale"] = _RULE_SCALE if c["rule"] else 0.0

    if c["kind"] in ("decode", "tokens"):
        # states of sequences that have run for a while: the last 64 tokens of a gated history (older ones have decayed)
        n = B * H
        s["H"], s["U"] = torch.empty((n, d, d), **f32), torch.empty((n, d, d), **f32)
        for i in range(0, n, 1024):
            m = min(1024, n - i)
            log_gate = torch.nn.functional.logsigmoid(normal(m, 64) + c["gate_mean"])
            weight = torch.exp(0.5 * (log_gate.sum(-1, keepdim=True) - log_gate.cumsum(-1)))[..., None]
            hk = rows(m, 64, d) * weight
            hv = normal(m, 64, d) * weight
            torch.bmm(hk.transpose(1, 2).contiguous(), hk, out=s["H"][i:i + m])
            torch.bmm(hv.transpose(1, 2).contiguous(), hk, out=s["U"][i:i + m])
        s["H"], s["U"] = s["H"].view(B, H, d, d), s["U"].view(B, H, d, d)
        s["layout"] = binding.GKA_STATE_H_LOWER_BLOCKS if c["lower"] else binding.GKA_STATE_FULL
        s["out"] = torch.empty_like(s["v"])
        return s
    io = binding.GKA_F32 if c["dtype"] == "f32" else binding.GKA_BF16
    compute = _COMPUTE[c["compute"]]
    if compute is None:
        compute = binding.GKA_COMPUTE_F32 if c["dtype"] == "f32" else binding.GKA_COMPUTE_BF16
    s["compute"] = compute
    some = s["gate"].data_ptr()              # (the size queries look at which options are in use, not at addresses)
    params = binding.make_params(B, H, T, d, c["r"], io, compute, lambda_scale=s["lambda_scale"],
                                 beta=some if c["beta"] else None, alpha=some if c["alpha"] else None)
    if c["kind"] == "forward":
        nbytes = binding.forward_workspace_bytes(params)
        s["out"] = torch.empty_like(s["v"])
    elif c["kind"] == "sketched":
        nbytes = binding.forward_sketched_workspace_bytes(params, c["d_s"])
        s["S"] = normal(H, c["d_s"], d) / d ** 0.5
        s["out"] = torch.empty_like(s["v"])
    else:
        nbytes = binding.backward_workspace_bytes(params)
        s["dy"] = normal(*lead, d).to(dt)
    s["workspace"] = torch.empty(max(nbytes, 256), dtype=torch.uint8, device="cuda")
    return s


def run(state):
    s, c = state, state["case"]
    options = dict(beta=s["beta"], alpha=s["alpha"], lambda_scale=s["lambda_scale"])
    if c["kind"] in ("decode", "tokens"):
        step = binding.gka_decode_step if c["kind"] == "decode" else binding.gka_decode_tokens
        o = step(s["H"], s["U"], s["q"], s["k"], s["v"], s["gate"], s["lam"], c["r"], out=s["out"],
                 state_layout=s["layout"], **options)
        return {"o": o, "H": s["H"], "U": s["U"]}
    if c["kind"] == "forward":
        got = binding.gka_forward(s["q"], s["k"], s["v"], s["gate"], s["lam"], c["r"], compute=s["compute"],
                                  return_state=c["states"], workspace=s["workspace"], out=s["out"], **options)
        return {"o": got[0], "H": got[1]["H_final"], "U": got[1]["U_final"]} if c["states"] else {"o": got}
    if c["kind"] == "sketched":
        return {"o": binding.gka_forward_sketched(s["q"], s["k"], s["v"], s["gate"], s["lam"], s["S"], c["r"],
                                                  beta=s["beta"], lambda_scale=s["lambda_scale"],
                                                  workspace=s["workspace"], out=s["out"])}
    return binding.gka_backward(s["q"], s["k"], s["v"], s["gate"], s["lam"], s["dy"], c["r"], compute=s["compute"],
                                workspace=s["workspace"], **options)


def _chunked(n, d_k, d_v, r, states, solves, readouts, forwards):
    """Multiply-adds of `n` tokens in chunks of 64, times two: `states` updates of d_k x d_v states, `forwards` Frobenius
    norms, `solves` runs of r passes in d_k dimensions, `readouts` of a d_k x d_v state (causal pairs only)."""
    pairs = 32.5                               # keys of its own chunk that an average token sees
    flops = states * 2 * d_k * d_v
    flops += forwards * (2 * d_k * d_k + 2 * pairs * d_k + 2 * pairs * 64)
    flops += solves * r * (2 * d_k * d_k + 4 * pairs * d_k)
    flops += readouts * (2 * d_k * d_v + 2 * pairs * (d_k + d_v))
    return n * flops


def work(case):
    c = _full(case)
    n, d, r = c["B"] * c["T"] * c["H"], c["d"], c["r"]
    esz = 4 if c["dtype"] == "f32" else 2
    scalars = 4 * n * (1 + (not c["rule"]) + c["beta"] + c["alpha"])
    state_bytes = 4 * d * d * c["B"] * c["H"]
    if c["kind"] in ("decode", "tokens"):
        h_part = (d // 32 + 1) / (2 * (d // 32)) if c["lower"] else 1.0
        return {"bytes": 2 * state_bytes * (1 + h_part) + 4 * n * d * esz + scalars,
                "flops": n * (2 * 3 * d * d + 2 * d * d + r * 2 * d * d + 2 * d * d)}
    if c["kind"] == "forward":
        if d <= 32:                           # a token at a time costs less there than chunks of 64 do
            flops = n * (2 * 3 * d * d + 2 * d * d + r * 2 * d * d + 2 * d * d)
        else:
            flops = _chunked(n, d, d, r, 2, 1, 1, 1)
        return {"bytes": 4 * n * d * esz + scalars + (2 * state_bytes if c["states"] else 0), "flops": flops}
    if c["kind"] == "sketched":
        d_s = c["d_s"]
        flops = n * 4 * d * d_s + _chunked(n, d_s, d_s, r, 1, 1, 0, 1) + _chunked(n, d_s, d, r, 1, 0, 1, 0)
        return {"bytes": 4 * n * d * esz + scalars + 4 * c["H"] * d_s * d, "flops": flops}
    # backward: two solves on one set of states, the forward readouts U^T dy and U xt and H x, and the readouts of the
    # two reverse recurrences (A k, A^T k, Ubar k, Ubar^T v); the rule adds H k and one more reverse recurrence
    grads = 3 * n * d * 4 + 4 * n * (1 + (not c["rule"]) + c["beta"] + c["alpha"])
    return {"bytes": 4 * n * d * esz + scalars + grads,
            "flops": _chunked(n, d, d, r, 4 + c["rule"], 2, 7 + 2 * c["rule"], 1)}


def tolerance(case):
    # About four times the 2-norm distance of today's results from a float64 evaluation of the same inputs (forward,
    # decode), or of the gradients from those with float32 products in the solves (backward):
    c = _full(case)
    if c["dtype"] == "f32":                       # 5e-7, float32 sums of some hundred terms
        return {"rel": 1e-5, "max": 1e-4}
    if c["kind"] in ("decode", "tokens") or c["d"] == 256:
        return {"rel": 6e-3, "max": 1.6e-2}       # 1.6e-3, max 3.9e-3: float32 arithmetic, the output rounded to bf16
    if c["kind"] == "backward":                   # 0.4e-2 - 0.8e-2 (max 0.08); with the rule 1.5e-2 - 2.6e-2 (max 0.11)
        return {"rel": 3e-2 if c["rule"] else 2e-2, "max": 0.4}
    if c["rule"]:                                 # 4.5e-3, max 0.056: condition number 51 at every token
        return {"rel": 1.8e-2, "max": 0.22}
    return {"rel": 1.2e-2, "max": 0.2}            # 3e-3, max 0.045: bf16 operands
