"""What a program does with this framework, as a list of measurable cases.

A case is one pass through the public entry points of
``paper_2507_02420_amd.gtt`` (and ``wtune``) on tensors that are on the GPU
already, with the plan that such a program keeps.  ``listed`` names the cases
that stand for real use, ``draw`` gives more of the same ranges, ``prepare``
makes the state a program has in hand before the call, ``run`` is the call,
``work`` the bytes and operations it cannot do without, and ``exact`` the
same results in 64 bits from plain torch.
"""
from __future__ import annotations

import math
import random

import torch

from paper_2507_02420_amd import gtt as G
from paper_2507_02420_amd import wtune

DTYPES = {"f64": torch.float64, "f32": torch.float32, "c128": torch.complex128, "c64": torch.complex64,
          "bf16": torch.bfloat16, "f16": torch.float16, "i32": torch.int32}
BYTES = {"f64": 8, "f32": 4, "c128": 16, "c64": 8, "bf16": 2, "f16": 2, "i32": 4}

# largest data a drawn case holds in one buffer (elements x bytes), half the
# largest listed one
MOST_BYTES = 1 << 28


def listed() -> list:
    return [
        # one vector, the smallest call: a state of ten qubits through the
        # Hadamard-like transform, where latency is all there is
        {"name": "vector_f64_b2_n10", "kind": "forward", "dtype": "f64", "b": 2, "n": 10, "batch": 1},
        # a small layer inside a model: forward and backward through autograd,
        # with the plan made by the call, a mini-batch of short vectors
        {"name": "autograd_f32_b4_n5_x32", "kind": "autograd", "dtype": "f32", "b": 4, "n": 5, "batch": 32},
        # integer Walsh-Hadamard transform of long vectors, exact mod 2^32
        {"name": "hadamard_i32_b2_n20_x16", "kind": "forward", "dtype": "i32", "b": 2, "n": 20, "batch": 16},
        # learning W by differentiation: the largest batch, forward keeping the
        # activations, then both gradients
        {"name": "train_c64_b8_n6_x256", "kind": "train", "dtype": "c64", "b": 8, "n": 6, "batch": 256},
        # the same for two-qubit blocks on long vectors: many digits a group
        {"name": "train_c64_b4_n10_x64", "kind": "train", "dtype": "c64", "b": 4, "n": 10, "batch": 64},
        # odd radix: lengths that are no multiple of a vector load
        {"name": "train_f32_b3_n13_x16", "kind": "train", "dtype": "f32", "b": 3, "n": 13, "batch": 16},
        # wide base matrix, 16-bit storage, matrix cores, both directions
        {"name": "train_bf16_b16_n4_x256", "kind": "train", "dtype": "bf16", "b": 16, "n": 4, "batch": 256},
        # distinct tensor factors, odd sizes, both directions
        {"name": "train_mixed_c64_x4096", "kind": "mixed", "dtype": "c64", "radices": "8,3,4,5,2,7", "batch": 4096},
        # serving: vectors of many lengths and radices in one call
        {"name": "ragged_bf16_x1024", "kind": "ragged", "dtype": "bf16", "count": 1024, "radices": "2,4,16,32",
         "least": 1 << 10, "most": 1 << 20, "shapes": 52},
        # natural-order filter: forward, split, two inverses
        {"name": "filter_c64_b4_n10_x64", "kind": "filter", "dtype": "c64", "b": 4, "n": 10, "batch": 64, "cutoff": 1 << 19},
        # state transmission: dominant coefficients of long vectors and the
        # receiver's reconstruction
        {"name": "topk_f32_b2_n20_x16", "kind": "topk", "dtype": "f32", "b": 2, "n": 20, "batch": 16, "k": 1 << 14},
        # one gradient of the tuning of W: kept energy, its gradient in W
        {"name": "wtune_c64_b8_n4_x256", "kind": "wtune", "dtype": "c64", "b": 8, "n": 4, "batch": 256, "k": 64},
    ]


def _log_int(rng: random.Random, lo: float, hi: float) -> int:
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _digits(rng: random.Random, b: int, lo: int, hi: int) -> int:
    """A digit count with lo <= b**n <= hi."""
    ns = [n for n in range(1, 32) if lo <= b ** n <= hi]
    return rng.choice(ns)


def draw(rng: random.Random) -> dict:
    kind = rng.choice(["forward", "forward", "autograd", "train", "train", "train", "mixed", "ragged", "filter", "topk",
                       "wtune"])
    if kind == "ragged":
        radices = rng.choice(["2,4,16,32", "2,4,16,32", "2,3,4,5,8"])
        return {"kind": kind, "dtype": rng.choice(["bf16", "bf16", "f16", "f32"]), "count": _log_int(rng, 9, 500),
                "radices": radices, "least": 1 << 10, "most": 1 << 20, "shapes": rng.randrange(1 << 20)}
    if kind == "mixed":
        m = rng.randint(2, 6)
        radices = [rng.randint(2, 8) for _ in range(m)]
        N = math.prod(radices)
        dtype = rng.choice(["c64", "c64", "f32"])
        batch = max(1, _log_int(rng, 1 << 18, MOST_BYTES / 2) // (N * BYTES[dtype]))
        return {"kind": kind, "dtype": dtype, "radices": ",".join(map(str, radices)), "batch": batch}
    if kind == "autograd":
        b = rng.choice([2, 3, 4, 5, 8, 16])
        return {"kind": kind, "dtype": rng.choice(["f32", "f32", "c64"]), "b": b, "n": _digits(rng, b, 1 << 6, 1 << 13),
                "batch": _log_int(rng, 4, 300)}
    if kind == "topk":
        b, n = 2, rng.randint(8, 20)
        batch = max(1, min(1000, _log_int(rng, 1 << 16, MOST_BYTES / 4) // (4 * 2 ** n)))
        return {"kind": kind, "dtype": rng.choice(["f32", "f32", "c64"]), "b": b, "n": n, "batch": batch,
                "k": max(1, _log_int(rng, 2 ** n / 128, 2 ** n / 16))}
    if kind == "wtune":
        b = rng.choice([2, 4, 8])
        n = _digits(rng, b, 1 << 8, 1 << 15)
        return {"kind": kind, "dtype": rng.choice(["c64", "c64", "f32"]), "b": b, "n": n,
                "batch": max(1, _log_int(rng, 1 << 16, 1 << 21) // b ** n), "k": rng.randint(3, b ** n // 8)}
    if kind == "filter":
        b = rng.choice([2, 4, 8])
        dtype = rng.choice(["c64", "c64", "f32"])
        n = _digits(rng, b, 1 << 8, 1 << 20)
        batch = max(1, _log_int(rng, 1 << 18, MOST_BYTES) // (BYTES[dtype] * b ** n))
        return {"kind": kind, "dtype": dtype, "b": b, "n": n, "batch": batch, "cutoff": rng.randint(1, b ** n - 1)}
    if kind == "forward":
        dtype = rng.choice(["f64", "f32", "c64", "i32", "bf16"])
        b = 2 if dtype == "i32" else rng.choice([2, 2, 4, 16, 32]) if dtype == "bf16" else rng.choice([2, 2, 3, 4, 5, 8])
        n = _digits(rng, b, 1 << 6, 1 << 20)
        batch = max(1, _log_int(rng, 1 << 13, MOST_BYTES) // (BYTES[dtype] * b ** n))
        return {"kind": kind, "dtype": dtype, "b": b, "n": n, "batch": batch}
    dtype = rng.choice(["c64", "c64", "f32", "f32", "bf16", "f16", "f64"])
    b = rng.choice([16, 32]) if dtype in ("bf16", "f16") else rng.choice([2, 3, 4, 5, 6, 7, 8, 16] if dtype == "f32" else
                                                                         [2, 3, 4, 5, 8])
    n = _digits(rng, b, 1 << 8, 1 << 20)
    batch = max(1, _log_int(rng, 1 << 18, MOST_BYTES / (1 if b in (2, 4, 8) else 4)) // (BYTES[dtype] * b ** n))
    return {"kind": "train", "dtype": dtype, "b": b, "n": n, "batch": batch,
            "fp32_intermediate": dtype in ("bf16", "f16") and rng.random() < 0.3}


# -- inputs -------------------------------------------------------------------
def _radices(case: dict) -> list:
    """The factors of one vector, most significant first."""
    if case["kind"] == "mixed":
        return [int(r) for r in case["radices"].split(",")]
    return [case["b"]] * case["n"]


def _length(case: dict) -> int:
    return math.prod(_radices(case))


def _shapes(case: dict) -> list:
    """(radix, digits) of every vector of a ragged batch."""
    rng = random.Random(case["shapes"])
    radices = [int(r) for r in case["radices"].split(",")]
    shapes = [(b, _digits(rng, b, case["least"], case["most"])) for b in (rng.choice(radices) for _ in range(case["count"]))]
    # every radix occurs, so that the table of matrices holds one of each
    return shapes[:max(0, len(shapes) - len(radices))] + [(b, _digits(rng, b, case["least"], case["most"])) for b in radices]


def _elements(case: dict) -> int:
    if case["kind"] == "ragged":
        return sum(b ** n for b, n in _shapes(case))
    return case["batch"] * _length(case)


def _unitary(b: int, is_complex: bool, gen: torch.Generator) -> torch.Tensor:
    """A random unitary (orthogonal) b x b matrix in 64 bits, on the host."""
    a = torch.randn(b, b, generator=gen, dtype=torch.complex128 if is_complex else torch.float64)
    q, r = torch.linalg.qr(a)
    d = torch.diagonal(r)
    return (q * (d / d.abs())).contiguous()


def _normal(shape, dtype: torch.dtype, gen: torch.Generator) -> torch.Tensor:
    made = torch.float32 if dtype in (torch.bfloat16, torch.float16) else dtype
    return torch.randn(shape, generator=gen, device="cuda", dtype=made).to(dtype)


def _planted(case: dict, W: torch.Tensor, gen: torch.Generator) -> torch.Tensor:
    """Vectors that k coefficients dominate, the kind that the transmission
    protocol and the tuning of W are for: magnitudes from 1 to 2 over a noise
    of 0.03."""
    dtype = DTYPES[case["dtype"]]
    wide = W.dtype
    N, batch = _length(case), case["batch"]
    c = 0.03 * torch.randn(batch, N, generator=gen, device="cuda", dtype=wide)
    at = torch.rand(batch, N, generator=gen, device="cuda").topk(case["k"], dim=1).indices
    big = torch.randn(batch, case["k"], generator=gen, device="cuda", dtype=wide)
    size = 1 + torch.rand(batch, case["k"], generator=gen, device="cuda", dtype=torch.float64)
    c.scatter_(1, at, big / big.abs() * size)
    return _apply(c, [W.conj().T.resolve_conj().contiguous()] * case["n"]).to(dtype)


def _inputs(case: dict, seed: int) -> dict:
    """W (one matrix, or several back to back) in the compute type, x, and gy
    for the kinds that differentiate."""
    host = torch.Generator().manual_seed(seed)
    gen = torch.Generator(device="cuda").manual_seed(seed)
    dtype = DTYPES[case["dtype"]]
    w_dtype = G.W_DTYPE[dtype]
    kind = case["kind"]
    if dtype == torch.int32:
        W = torch.tensor([[1, 1], [1, -1]], dtype=torch.int32, device="cuda")
        x = torch.randint(-100, 101, (case["batch"], _length(case)), generator=gen, device="cuda", dtype=torch.int32)
        return {"W": W, "x": x}
    if kind == "ragged":
        radices = sorted({b for b, _ in _shapes(case)})
        W = torch.cat([_unitary(b, dtype.is_complex, host).reshape(-1) for b in radices]).cuda().to(w_dtype)
        return {"W": W, "x": _normal((_elements(case),), dtype, gen)}
    if kind == "mixed":
        W = torch.cat([_unitary(b, dtype.is_complex, host).reshape(-1) for b in _radices(case)]).cuda().to(w_dtype)
    else:
        W = _unitary(case["b"], dtype.is_complex, host).cuda().to(w_dtype)
    if kind in ("topk", "wtune"):
        return {"W": W, "x": _planted(case, W.to(torch.complex128 if dtype.is_complex else torch.float64), gen)}
    got = {"W": W, "x": _normal((case["batch"], _length(case)), dtype, gen)}
    if kind in ("train", "mixed", "autograd"):
        got["gy"] = _normal((case["batch"], _length(case)), dtype, gen)
    return got


def prepare(case: dict, seed: int) -> dict:
    state = {"case": case, **_inputs(case, seed)}
    kind, dtype = case["kind"], DTYPES[case["dtype"]]
    if kind == "autograd":
        state["W"].requires_grad_()
        state["x"].requires_grad_()
        return state
    if kind == "ragged":
        shapes = _shapes(case)
        state["plan"] = G.Plan([b for b, _ in shapes], [n for _, n in shapes], dtype=dtype)
    elif kind == "mixed":
        state["plan"] = G.Plan.mixed(_radices(case), case["batch"], dtype)
    else:
        flags = G.FLAG_FP32_INTERMEDIATE if case.get("fp32_intermediate") else 0
        state["plan"] = G.Plan(case["b"], case["n"], case["batch"], dtype, flags)
    if kind in ("train", "mixed"):
        # a training loop keeps its buffers
        saved = state["plan"].workspace_size()[2]
        state["saved"] = torch.empty(saved, dtype=torch.uint8, device="cuda") if saved else None
        state["y"], state["gx"] = torch.empty_like(state["x"]), torch.empty_like(state["x"])
        state["gW"] = torch.empty_like(state["W"])
    return state


def run(state: dict):
    case, W, x, plan = state["case"], state["W"], state["x"], state.get("plan")
    kind = case["kind"]
    if kind in ("forward", "ragged"):
        return plan.forward(W, x)
    if kind == "autograd":
        y = G.gtt(x, W, case["b"], case["n"])
        gx, gW = torch.autograd.grad(y, (x, W), state["gy"])
        return y, gx, gW
    if kind in ("train", "mixed"):
        y = plan.forward(W, x, state["y"], saved=state["saved"])
        gx, gW = plan.backward(W, x, state["gy"], saved=state["saved"], gx=state["gx"], gW=state["gW"])
        return y, gx, gW
    if kind == "filter":
        return plan.filter(W, x, case["cutoff"])
    if kind == "topk":
        return plan.compress(W, x, case["k"])
    energy, idx, val = wtune.kept_energy(plan, W, x, case["k"])
    gy = torch.zeros_like(x)
    gy.scatter_(1, idx, 2 * val)
    _, gW = plan.backward(W, x, gy, want_gx=False)
    return energy, idx, val, gW


def work(case: dict) -> dict:
    E, size = _elements(case), BYTES[case["dtype"]]
    mul = 8 if case["dtype"] in ("c64", "c128") else 2
    kind = case["kind"]
    # multiply-adds of one transform: every element, every digit, b terms
    if kind == "ragged":
        one = sum(mul * b * n * b ** n for b, n in _shapes(case))
    else:
        one = mul * sum(_radices(case)) * E
    if kind in ("forward", "ragged"):
        return {"bytes": 2 * E * size, "flops": one}
    if kind in ("train", "mixed", "autograd"):
        # reads x and gy, writes y and gx; the transform, its adjoint and the
        # products of the gradient of W
        return {"bytes": 4 * E * size, "flops": 3 * one}
    if kind == "filter":
        return {"bytes": 3 * E * size, "flops": 3 * one}
    kept = case["batch"] * case["k"] * (8 + size)
    if kind == "topk":
        return {"bytes": 2 * E * size + kept, "flops": 2 * one}
    return {"bytes": E * size + kept, "flops": 3 * one}


# -- the same in 64 bits --------------------------------------------------------
def _wide(t: torch.Tensor) -> torch.Tensor:
    return t.detach().to(torch.complex128 if t.is_complex() else torch.float64)


def _apply(x: torch.Tensor, factors: list, kept: list = None) -> torch.Tensor:
    """(factors[0] kron factors[1] kron ...) x for rows x, one digit at a time
    from the least significant: each pass multiplies by the last axis' factor
    and moves that axis to the front.  `kept` receives each pass's input and
    the radix's position, as rows of one digit."""
    rows = x.shape[0]
    for W in reversed(factors):
        b = W.shape[0]
        a = x.reshape(-1, b)
        if kept is not None:
            kept.append(a)
        x = (a @ W.T.contiguous()).reshape(rows, -1, b).transpose(1, 2).reshape(rows, -1)
    return x


def _grads(x: torch.Tensor, gy: torch.Tensor, factors: list):
    """y, gx and the gradient of every factor."""
    kept = []
    y = _apply(x, factors, kept)
    rows, c, gW = x.shape[0], gy, [None] * len(factors)
    for k, W in enumerate(factors):
        b = W.shape[0]
        c = c.reshape(rows, b, -1).transpose(1, 2).reshape(-1, b)
        a = kept.pop().conj()
        gW[k] = torch.stack([(c[:, r:r + 1] * a).sum(0) for r in range(b)])
        c = (c @ W.conj().resolve_conj()).reshape(rows, -1)
    return y, c, gW


def exact(case: dict, seed: int):
    if case["dtype"] == "i32":
        return None
    t = _inputs(case, seed)
    kind, W, x = case["kind"], _wide(t["W"]), _wide(t["x"])
    if kind == "ragged":
        shapes = _shapes(case)
        radices = sorted({b for b, _ in shapes})
        table, at = {}, 0
        for b in radices:
            table[b] = W[at:at + b * b].reshape(b, b)
            at += b * b
        y, at = torch.empty_like(x), 0
        for b, n in shapes:
            y[at:at + b ** n] = _apply(x[at:at + b ** n].reshape(1, -1), [table[b]] * n)[0]
            at += b ** n
        return y
    if kind == "mixed":
        factors, at = [], 0
        for b in _radices(case):
            factors.append(W[at:at + b * b].reshape(b, b))
            at += b * b
    else:
        factors = [W] * case["n"]
    if kind == "forward":
        return _apply(x, factors)
    if kind in ("train", "mixed", "autograd"):
        y, gx, gW = _grads(x, _wide(t["gy"]), factors)
        return y, gx, torch.cat([g.reshape(-1) for g in gW]) if kind == "mixed" else sum(gW)
    adjoint = [F.conj().T.resolve_conj().contiguous() for F in factors]
    y = _apply(x, factors)
    if kind == "filter":
        low, high = y.clone(), y.clone()
        low[:, case["cutoff"]:] = 0
        high[:, :case["cutoff"]] = 0
        return _apply(low, adjoint), _apply(high, adjoint)
    idx = y.abs().topk(case["k"], dim=1).indices.sort(dim=1).values
    val = y.gather(1, idx)
    only = torch.zeros_like(y).scatter_(1, idx, val)
    if kind == "topk":
        return idx, val, _apply(only, adjoint)
    return float(val.abs().square().sum()), idx, val, sum(_grads(x, 2 * only, factors)[2])
