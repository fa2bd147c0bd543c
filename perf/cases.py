"""Workloads of FLuRKA attention for timing, as a program that uses the library runs them.

A case is a dict of plain values: the entry points it goes through (`pass`), the tensor sizes, the
storage type, the feature map and the options.  `prepare` draws its inputs on the GPU, `run` makes one
pass through the public binding, `work` counts the bytes and operations the method itself needs.

Distributions are the benchmark recipe's (paper_2306_15799_amd/inputs.py): Q, K, V ~ N(0, 1) d^(-1/4);
E, F ~ N(0, 1/k); omega, dOut ~ N(0, 1); paper-order inputs X ~ N(0, 1), W ~ N(0, 1/dm) d^(-1/4).
"""
import math

import torch

from paper_2306_15799_amd import binding as fb
from paper_2306_15799_amd.inputs import DERIVED_WORKLOADS, PHI_ELU1, PHI_PERFORMER, WORKLOADS

# `pass` of a case
FORWARD = "forward"          # flurka_attn_fwd: inference
TRAIN = "train"              # flurka_attn_fwd + flurka_attn_bwd: one training step of the layer
PAPER_ORDER = "paper_order"  # flurka_attn_fwd_fused_w: projection of the layer input, then the transforms
VARIANT = "variant"          # flurka_attn_fwd_ex + flurka_attn_bwd_ex: one projection pair per head,
#                              float32 dE / dF, gradient for omega


def _case(passes, B, H, n, d, k, m, dtype="bf16", phi=PHI_PERFORMER, name=None, **more):
    c = {"pass": passes, "B": B, "H": H, "n": n, "d": d, "k": k, "m": d if phi == PHI_ELU1 else m,
         "dtype": dtype, "phi": phi, **more}
    if name:
        c["name"] = name
    return c


def _workload(name, w):
    return _case(TRAIN if w.backward else FORWARD, w.B, w.H, w.n, w.d, w.k, w.m, w.dtype, w.phi, name)


def listed():
    return [
        # one short fp32 sequence, one head: the smallest call, all latency and launches
        _workload("c1_forward_f32", WORKLOADS["C1"]),
        # a small bf16 training step (a short-sequence layer, a unit test, a first batch): launches again
        _case(TRAIN, 2, 2, 512, 64, 64, 64, name="small_train"),
        # encoder inference at batch 8: an ordinary sequence length
        _workload("c2_forward", WORKLOADS["C2"]),
        # the elu map at long sequences, inference and as a training step
        _workload("c3_forward_elu", WORKLOADS["C3"]),
        _workload("c3_train_elu", DERIVED_WORKLOADS["C3T"]),
        # one very long sequence, wide heads: inference and the training step (the largest case)
        _workload("c4_forward_long", WORKLOADS["C4"]),
        _workload("c4_train_long", DERIVED_WORKLOADS["C4T"]),
        # the headline training step
        _workload("c5_train", WORKLOADS["C5"]),
        # a training step on unpadded text: a sequence length, key count and feature count that no tile divides
        _case(TRAIN, 4, 12, 3001, 64, 187, 150, name="ragged_train"),
        # a training step in full precision (finding out whether bf16 is to blame)
        _case(TRAIN, 2, 8, 4096, 64, 256, 256, dtype="f32", name="f32_train"),
        # a training step with everything trainable: per-head projections, float32 dE / dF, omega's gradient
        _case(VARIANT, 2, 8, 2048, 64, 128, 128, name="variant_train"),
        # the layer input projected before the per-head transforms, at the sweep's sequence length
        _case(PAPER_ORDER, 1, 16, 20032, 64, 512, 256, dm=1024, name="paper_order_forward"),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    """One more case of the ranges the listed ones stand for."""
    kind = rng.choices(["forward", "train", "elu", "ragged", "f32", "variant", "paper_order"],
                       weights=[20, 28, 14, 14, 10, 6, 8])[0]
    B, H = rng.choice([1, 1, 2, 3, 4, 8]), rng.choice([1, 2, 4, 6, 8, 12, 16])
    k = _log_int(rng, 32, 512)
    m = rng.choice([32, 64, 96, 128, 192, 256, _log_int(rng, 16, 256)])
    phi = PHI_PERFORMER

    def length(lo, hi, per_key, elements):
        """A sequence length in lo..hi with at most `per_key` positions per projected key (the keys' norms
        grow with that ratio) and at most `elements` elements in a (B, H, n, d) tensor."""
        return _log_int(rng, lo, max(lo + 1, min(hi, per_key * k, elements // (B * H * d))))

    if kind == "forward":            # lengths that are multiples of 8, as a padded batch has them
        d = rng.choice([64, 64, 128])
        n = length(256, 65536, 128, 1 << 27) // 8 * 8
        return _case(FORWARD, B, H, n, d, k, m, phi=phi)
    if kind == "train":
        d = rng.choice([64, 64, 128])
        n = length(256, 20480, 40, 1 << 26) // 32 * 32
        return _case(TRAIN, B, H, n, d, k, m, phi=phi)
    if kind == "elu":
        d = rng.choice([64, 64, 128])
        n = length(256, 32768, 128, 1 << 26) // 32 * 32
        return _case(rng.choice([FORWARD, TRAIN]), B, H, n, d, k, m, phi=PHI_ELU1)
    if kind == "ragged":             # any length, key count and feature count; other head sizes as well
        d = rng.choice([64, 64, 64, 128, 32, 80, 96])
        n = length(200, 8192, 40, 1 << 24)
        return _case(rng.choice([FORWARD, TRAIN, TRAIN]), B, H, n, d, k, m,
                     phi=rng.choice([PHI_PERFORMER, PHI_PERFORMER, PHI_ELU1]))
    if kind == "f32":
        d = rng.choice([32, 64, 64, 128])
        n = length(200, 8192, 16, 1 << 23)
        return _case(rng.choice([FORWARD, TRAIN]), B, H, n, d, k, m, dtype="f32",
                     phi=rng.choice([PHI_PERFORMER, PHI_PERFORMER, PHI_ELU1]))
    if kind == "variant":
        d = rng.choice([32, 64, 64, 128])
        n = length(200, 8192, 40, 1 << 22)
        return _case(VARIANT, B, H, n, d, k, m)
    d = rng.choice([64, 64, 128])    # paper order
    H = rng.choice([4, 8, 16, 32])
    B = rng.choice([1, 1, 2])
    n = length(512, 32768, 64, 1 << 26) // 8 * 8
    return _case(PAPER_ORDER, B, H, n, d, k, m, dm=H * d)


def prepare(case, seed):
    c = case
    dev = torch.device("cuda")
    td = torch.bfloat16 if c["dtype"] == "bf16" else torch.float32
    gen = torch.Generator(device=dev).manual_seed(seed)

    def normal(shape, scale=1.0):
        return torch.randn(shape, generator=gen, device=dev, dtype=torch.float32).mul_(scale).to(td)

    B, H, n, d, k, m = (c[x] for x in ("B", "H", "n", "d", "k", "m"))
    qkv, ef = float(d) ** -0.25, float(k) ** -0.5
    s = {"case": c, "Q": normal((B, H, n, d), qkv)}
    if c["pass"] == PAPER_ORDER:
        dm = c["dm"]
        s["XK"], s["XV"] = normal((B, n, dm)), normal((B, n, dm))
        s["WK"], s["WV"] = (normal((H, d, dm), qkv * float(dm) ** -0.5) for _ in range(2))
    else:
        s["K"], s["V"] = normal((B, H, n, d), qkv), normal((B, H, n, d), qkv)
    ef_shape = (H, k, n) if c["pass"] == VARIANT else (k, n)
    s["E"], s["F"] = normal(ef_shape, ef), normal(ef_shape, ef)
    s["omega"] = normal((H, m, d)) if c["phi"] == PHI_PERFORMER else None
    if c["pass"] in (TRAIN, VARIANT):
        s["dOut"] = normal((B, H, n, d))
    return s


def run(state):
    s = state
    c = s["case"]
    phi = c["phi"]
    if c["pass"] == PAPER_ORDER:
        out, _ = fb.flurka_attn_fwd_fused_w(s["Q"], s["XK"], s["XV"], s["E"], s["F"], s["WK"], s["WV"], s["omega"], phi=phi)
        return out
    inputs = (s["Q"], s["K"], s["V"], s["E"], s["F"], s["omega"])
    if c["pass"] == VARIANT:
        out, ctx = fb.flurka_attn_fwd_ex(*inputs, phi=phi, ef_per_head=True)
        grads = fb.flurka_attn_bwd_ex(*inputs, out, s["dOut"], ctx, phi=phi, ef_per_head=True, grad_ef_f32=True,
                                      want_d_omega=True)
        return (out, *grads)
    out, ctx = fb.flurka_attn_fwd(*inputs, phi=phi)
    if c["pass"] == FORWARD:
        return out
    grads = fb.flurka_attn_bwd(*inputs, out, s["dOut"], ctx, phi=phi)
    return (out, *grads)


def work(case):
    """Every input read once, every result written once; the contractions of the method (associative
    order), the query features formed again by the backward pass."""
    c = case
    B, H, n, d, k, m = (c[x] for x in ("B", "H", "n", "d", "k", "m"))
    es = 2 if c["dtype"] == "bf16" else 4
    performer = c["phi"] == PHI_PERFORMER
    row = B * H * n * d                      # elements of Q, and of each tensor like it
    pair = 2 * k * n * (H if c["pass"] == VARIANT else 1)      # elements of E and F
    omega = H * m * d if performer else 0
    features = 2 * row * m if performer else 0                 # omega q; the elu map contracts nothing
    key = 2 * B * H * k * m * d * ((2 if performer else 1))    # features of K', then PhiK^T V'
    if c["pass"] == PAPER_ORDER:
        dm = c["dm"]
        return {"bytes": es * (2 * row + 2 * B * n * dm + 2 * H * d * dm + pair + omega),
                "flops": 4 * B * k * n * dm + 4 * B * H * k * dm * d + key + features + 2 * row * m}
    forward = {"bytes": es * (4 * row + pair + omega), "flops": 4 * row * k + key + features + 2 * row * m}
    if c["pass"] == FORWARD:
        return forward
    # backward: G S^T, the query gradient and dS over n; four products on the key side; dK, dV, dE, dF
    flops = features + 2 * row * m * (3 if performer else 2) + 2 * key + 8 * row * k
    grads = es * (3 * row)
    if c["pass"] == VARIANT:
        grads += 4 * (pair + omega)
        flops += 2 * row * m + key // 2      # d omega
    else:
        grads += es * pair
    return {"bytes": forward["bytes"] + es * row + grads, "flops": forward["flops"] + flops}


def tolerance(case):
    """About four times the error of the present code against the same formulas in float64 with automatic
    differentiation, over the listed cases and 120 drawn ones.  bf16: at most 3.6e-3 (dK, dE; 1.7e-3 is the
    rounding of a bf16 result), single values up to 0.11 of the larger of value and root mean square.
    f32: 3.6e-6 and 7e-5 (key exponents in the hundreds, taken to the exponential)."""
    return {"rel": 1.2e-2, "max": 0.4} if case["dtype"] == "bf16" else {"rel": 1.5e-5, "max": 3e-4}
