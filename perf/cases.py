"""The work a program has this library do, as timed cases.

Sizes are those of LLaMA layers at the ranks of the bench's sweep (a 4096-wide
attention projection, the 4096 -> 11008 MLP projections, the 8192 -> 28672 up
projection), ragged row counts and odd ranks beside the round ones, and both
directions: decode and prefill, forward and backward, plus the steps that make
a layer (calibration sums, reconstruction, pivoting factorization).  Values are
synthetic with the scales of a rank-r product of Gaussian factors.
"""
from __future__ import annotations

import math

import torch

from paper_2501_19090_amd import pifa

DEVICE = "cuda"
LAM, ALPHA = 0.25, 0.001  # the method's mix ratio and regularisation

# Largest product a drawn case may ask for: 2 * 4096 * 4096 * (8192 + 28672 - 4096).
MAX_FLOPS = 1.1e12


def listed():
    return [
        # one token through one attention projection: two launches over 25 MB of weights
        {"name": "decode_attn_m1", "kind": "forward", "d_in": 4096, "d_out": 4096, "r": 2048, "m": 1, "dtype": "bf16"},
        # one token through the largest projection: 269 MB of weights, past every cache
        {"name": "decode_up28672_m1", "kind": "forward", "d_in": 8192, "d_out": 28672, "r": 4096, "m": 1,
         "dtype": "bf16"},
        # eight concurrent sequences through an MLP's gate and up projections at once
        {"name": "decode_gate_up_m8", "kind": "group", "d_in": 4096, "d_outs": "11008,11008", "rs": "2048,2048",
         "m": 8},
        # a batch of decoding sequences, or a short prompt: a ragged handful of rows
        {"name": "batch_attn_m100", "kind": "forward", "d_in": 4096, "d_out": 4096, "r": 2048, "m": 100,
         "dtype": "bf16"},
        # the prompt of a LLaMA-7B-sized attention projection
        {"name": "prefill_attn_m4096", "kind": "forward", "d_in": 4096, "d_out": 4096, "r": 2048, "m": 4096,
         "dtype": "bf16"},
        # an MLP projection at a per-module rank, with a ragged prompt
        {"name": "prefill_up_r2867_m1999", "kind": "forward", "d_in": 4096, "d_out": 11008, "r": 2867, "m": 1999,
         "dtype": "bf16"},
        # the prompt of the largest projection
        {"name": "prefill_up28672_m4096", "kind": "forward", "d_in": 8192, "d_out": 28672, "r": 4096, "m": 4096,
         "dtype": "bf16"},
        # fine-tuning: every gradient of an attention projection
        {"name": "backward_attn_m4096", "kind": "backward", "d_in": 4096, "d_out": 4096, "r": 2048, "m": 4096},
        # a full-precision layer
        {"name": "f32_attn_m1024", "kind": "forward", "d_in": 4096, "d_out": 4096, "r": 2048, "m": 1024,
         "dtype": "f32"},
        # a layer's calibration sums over eight batches of 2048 tokens
        {"name": "calibrate_4096", "kind": "calibrate", "d_in": 4096, "batch": 2048, "batches": 8},
        # the closed-form U and V updates from those sums
        {"name": "reconstruct_4096", "kind": "reconstruct", "d_in": 4096, "d_out": 4096, "r": 2048},
        # pivoting factorization of one low-rank weight
        {"name": "build_4096", "kind": "build", "d_in": 4096, "d_out": 4096, "r": 2048},
    ]


def _logint(rng, lo, hi, step=1):
    return min(hi, max(lo, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi))) / step)) * step))


def _rank(rng, d_in, d_out):
    return max(1, int(rng.uniform(0.1, 0.9) * min(d_in, d_out)))


def draw(rng):
    kind = rng.choice(["forward", "forward", "forward", "forward", "forward_f32", "group", "group", "backward",
                       "backward", "calibrate", "reconstruct", "build"])
    if kind == "calibrate":
        return {"kind": kind, "d_in": _logint(rng, 512, 8192, 8), "batch": _logint(rng, 128, 4096),
                "batches": rng.randint(1, 8)}
    if kind in ("reconstruct", "build"):
        d_in, d_out = _logint(rng, 256, 4096, 8), _logint(rng, 256, 4096)
        return {"kind": kind, "d_in": d_in, "d_out": d_out, "r": max(1, int(rng.uniform(0.1, 0.5) * min(d_in, d_out)))}
    f32 = kind == "forward_f32"
    d_in = _logint(rng, 256, 4096 if f32 else 8192, 8)
    m = _logint(rng, 64 if kind == "backward" else 1, 2048 if f32 else 8192)
    if kind == "group":
        n = rng.randint(2, 3)
        d_outs = [_logint(rng, 256, 11008) for _ in range(n)]
        rs = [_rank(rng, d_in, d) for d in d_outs]
        m = min(m, 4096)
        return {"kind": kind, "d_in": d_in, "d_outs": ",".join(map(str, d_outs)), "rs": ",".join(map(str, rs)), "m": m}
    d_out = _logint(rng, 256, 4096 if f32 else 11008)
    r = _rank(rng, d_in, d_out)
    per_row = 2.0 * r * (d_in + d_out - r) * (3 if kind == "backward" else 1)
    m = max(1, min(m, int((2e11 if f32 else MAX_FLOPS) / per_row)))
    if kind == "backward":
        return {"kind": kind, "d_in": d_in, "d_out": d_out, "r": r, "m": m}
    return {"kind": "forward", "d_in": d_in, "d_out": d_out, "r": r, "m": m, "dtype": "f32" if f32 else "bf16"}


# ------------------------------------------------------------------ inputs
def _generator(seed):
    g = torch.Generator(device=DEVICE)
    g.manual_seed(int(seed) * 7919 + 17)
    return g


def _randn(g, *shape, scale=1.0, dtype=torch.float32):
    work = torch.float64 if dtype == torch.float64 else torch.float32
    return (torch.randn(*shape, generator=g, device=DEVICE, dtype=work) * scale).to(dtype)


def _partition(g, d_out, r):
    perm = torch.randperm(d_out, generator=g, device=DEVICE)
    return torch.sort(perm[:r])[0], torch.sort(perm[r:])[0]


def _layer(g, d_in, d_out, r, dtype):
    """Pivot rows with the scale of a product of N(0, 1/r) factors, and
    coefficients that give the non-pivot outputs the pivot outputs' scale."""
    piv, npiv = _partition(g, d_out, r)
    Wp = _randn(g, r, d_in, scale=r ** -0.5, dtype=dtype)
    C = _randn(g, d_out - r, r, scale=r ** -0.5, dtype=dtype)
    return Wp, C, piv, npiv


def _forward64(X, Wp, C, piv, npiv, d_out):
    Yp = X.double() @ Wp.double().t()
    Y = torch.empty((X.shape[0], d_out), dtype=torch.float64, device=X.device)
    Y[:, piv] = Yp
    Y[:, npiv] = Yp @ C.double().t()
    return Y


def _dtype(case):
    return torch.float32 if case.get("dtype") == "f32" else torch.bfloat16


def _members(case):
    return [(int(d), int(r)) for d, r in zip(case["d_outs"].split(","), case["rs"].split(","))]


def _inputs(case, seed):
    """Device inputs of a case, from the seed alone."""
    g = _generator(seed)
    kind = case["kind"]
    d_in = case["d_in"]
    if kind == "group":
        layers = [_layer(g, d_in, d, r, torch.bfloat16) for d, r in _members(case)]
        return {"layers": layers, "X": _randn(g, case["m"], d_in, dtype=torch.bfloat16)}
    if kind in ("forward", "backward"):
        dt = _dtype(case)
        layer = _layer(g, d_in, case["d_out"], case["r"], dt)
        out = {"layer": layer, "X": _randn(g, case["m"], d_in, dtype=dt)}
        if kind == "backward":
            out["Y"] = _forward64(out["X"], *layer, case["d_out"]).to(torch.bfloat16)
            out["dY"] = _randn(g, case["m"], case["d_out"], scale=1e-2, dtype=torch.bfloat16)
        return out
    if kind == "calibrate":
        Xo = [_randn(g, case["batch"], d_in, dtype=torch.bfloat16) for _ in range(case["batches"])]
        # the low-rank flow's activations: the dense flow's with some error on top
        Xu = [(x.float() + 0.1 * _randn(g, *x.shape)).to(torch.bfloat16) for x in Xo]
        return {"Xo": Xo, "Xu": Xu}
    d_out, r = case["d_out"], case["r"]
    U = _randn(g, d_out, r, scale=r ** -0.5, dtype=torch.float64)
    V = _randn(g, r, d_in, scale=r ** -0.5, dtype=torch.float64)
    if kind == "build":
        return {"W": U @ V, "U": U}
    W = U @ V + _randn(g, d_out, d_in, scale=0.3 * r ** -0.5, dtype=torch.float64)
    tokens = 2 * d_in
    Xo = _randn(g, tokens, d_in, dtype=torch.bfloat16)
    Xu = (Xo.float() + 0.1 * _randn(g, tokens, d_in)).to(torch.bfloat16)
    return {"W": W, "Vt": V, "Xo": Xo, "Xu": Xu}


class _Handle:
    """Gives a handle back when the state goes."""

    def __init__(self, handle, destroy):
        self.handle, self.destroy = handle, destroy

    def __del__(self):
        if self.handle:
            self.destroy(self.handle)
            self.handle = 0


def _host(idx):
    return idx.to(torch.int32).cpu().numpy()


def prepare(case, seed):
    kind, d_in = case["kind"], case["d_in"]
    src = _inputs(case, seed)
    if kind == "group":
        specs = [(Wp, C, _host(p), _host(n), (d_in, d, r))
                 for (Wp, C, p, n), (d, r) in zip(src["layers"], _members(case))]
        Y = torch.empty((case["m"], sum(d for d, _ in _members(case))), dtype=torch.bfloat16, device=DEVICE)
        owner = _Handle(pifa.pifa_group_create(specs), pifa.pifa_group_destroy)
        return {"kind": kind, "owner": owner, "X": src["X"], "Y": Y}
    if kind in ("forward", "backward"):
        Wp, C, piv, npiv = src["layer"]
        layer = pifa.PifaLayer(Wp, C, _host(piv), _host(npiv), case["d_out"])
        if kind == "forward":
            Y = torch.empty((case["m"], case["d_out"]), dtype=_dtype(case), device=DEVICE)
            return {"kind": kind, "layer": layer, "X": src["X"], "Y": Y}
        r = case["r"]
        return {"kind": kind, "layer": layer, "X": src["X"], "Y": src["Y"], "dY": src["dY"],
                "dX": torch.empty_like(src["X"]),
                "dWp": torch.empty((r, d_in), dtype=torch.float32, device=DEVICE),
                "dC": torch.empty((case["d_out"] - r, r), dtype=torch.float32, device=DEVICE)}
    if kind == "build":
        return {"kind": kind, "W": src["W"], "r": case["r"]}
    owner = _Handle(pifa.pifa_calib_create(d_in), pifa.pifa_calib_destroy)
    if kind == "calibrate":
        S = torch.empty((d_in, d_in), dtype=torch.float64, device=DEVICE)
        return {"kind": kind, "owner": owner, "Xo": src["Xo"], "Xu": src["Xu"], "S": S, "P": torch.empty_like(S)}
    pifa.pifa_calib_accumulate(owner.handle, src["Xo"], src["Xu"])
    r = case["r"]
    return {"kind": kind, "owner": owner, "W": src["W"], "Vt": src["Vt"],
            "U_r": torch.empty((case["d_out"], r), dtype=torch.float64, device=DEVICE),
            "Vt_r": torch.empty((r, d_in), dtype=torch.float64, device=DEVICE)}


def run(state):
    kind = state["kind"]
    if kind == "forward":
        return state["layer"](state["X"], state["Y"])
    if kind == "group":
        pifa.pifa_group_forward(state["owner"].handle, state["X"], state["Y"])
        return state["Y"]
    if kind == "backward":
        pifa.pifa_layer_backward(state["layer"].handle, state["X"], state["Y"], state["dY"], state["dX"],
                                 state["dWp"], state["dC"])
        return {"dX": state["dX"], "dWp": state["dWp"], "dC": state["dC"]}
    if kind == "calibrate":
        handle = state["owner"].handle
        pifa.pifa_calib_reset(handle)
        for xo, xu in zip(state["Xo"], state["Xu"]):
            pifa.pifa_calib_accumulate(handle, xo, xu)
        pifa.pifa_calib_read(handle, state["S"], state["P"])
        return {"S": state["S"], "P": state["P"]}
    if kind == "reconstruct":
        U_r, Vt_r = pifa.pifa_calib_reconstruct(state["owner"].handle, state["W"], state["Vt"], LAM, ALPHA,
                                                state["U_r"], state["Vt_r"])
        return {"U_r": U_r, "Vt_r": Vt_r}
    piv, npiv, Wp, C, report = pifa.pifa_build_f64(state["W"], state["r"])
    return {"piv": piv, "npiv": npiv, "Wp": Wp, "C": C, "report": report}


def work(case):
    kind, n = case["kind"], case["d_in"]
    if kind == "group":
        m, mem = case["m"], _members(case)
        weights = sum(r * n + (d - r) * r for d, r in mem)
        outs = sum(d for d, _ in mem)
        return {"bytes": 2 * weights + 4 * outs + 2 * m * (n + outs), "flops": 2 * m * weights}
    if kind == "calibrate":
        tokens = case["batch"] * case["batches"]
        # S is symmetric: half of its products; both sums written once in fp64
        return {"bytes": 2 * 2 * tokens * n + 2 * 8 * n * n, "flops": 3 * tokens * n * n}
    d, r = case["d_out"], case["r"]
    if kind == "build":
        # Householder QR of r steps on n x d, then the triangular solve for C
        qr = sum(4.0 * (n - k) * (d - k) for k in range(r))
        return {"bytes": 8 * (d * n + r * n + (d - r) * r), "flops": int(qr + (d - r) * r * r)}
    if kind == "reconstruct":
        products = 2.0 * (d * n * n + n * r * n + r * r * n + r * d * n + r * r * d + r * n * d)
        solves = r ** 3 / 3.0 * 2 + n ** 3 / 3.0 + 2.0 * r * r * (d + n) + 2.0 * n * n * r
        return {"bytes": 8 * (2 * n * n + d * n + r * n + d * r + r * n), "flops": int(products + solves)}
    m, es = case["m"], 4 if case.get("dtype") == "f32" else 2
    weights = r * n + (d - r) * r
    if kind == "backward":
        return {"bytes": 2 * (weights + m * n + 2 * m * d + m * n) + 4 * weights,
                "flops": 2 * m * r * (2 * (d - r) + 2 * n)}
    return {"bytes": es * weights + 4 * d + es * m * (n + d), "flops": 2 * m * weights}


def tolerance(case):
    """About four times the error against 64-bit sums that the path shows: bf16
    outputs 1.7e-3 (their rounding), fp32 layers 1.3e-6, calibration sums
    1.6e-7 (fp32 within a batch, fp64 across), the reconstruction of those sums
    5e-7, the fp64 factorization 1.3e-13 (more for worse conditioned rows)."""
    kind = case["kind"]
    if kind in ("forward", "group", "backward"):
        return {"rel": 5e-6 if case.get("dtype") == "f32" else 7e-3}
    return {"rel": {"calibrate": 1e-6, "reconstruct": 2e-6, "build": 1e-10}[kind]}


# ------------------------------------------------------------------ reference
def _pivoted_rows(W, r):
    """The r rows picked by QR with column pivoting on W^T (largest residual
    norm, ties to the lowest row), and the diagonal of R."""
    A = W.clone()  # row j holds what is left of row j
    left = torch.arange(W.shape[0], device=W.device)
    norms = (A * A).sum(1)
    alive = torch.ones(W.shape[0], dtype=torch.bool, device=W.device)
    picked, diag = [], []
    for _ in range(r):
        j = torch.argmax(torch.where(alive, norms, -1.0))
        v = A[j]
        d = torch.sqrt((v * v).sum())
        q = v / d
        A = torch.addr(A, A @ q, q, alpha=-1.0)
        norms = (A * A).sum(1)
        alive[j] = False
        picked.append(left[j])
        diag.append(d)
    return torch.stack(picked), torch.stack(diag)


def exact(case, seed):
    kind = case["kind"]
    src = _inputs(case, seed)
    if kind == "group":
        ys = [_forward64(src["X"], *layer, d) for layer, (d, _) in zip(src["layers"], _members(case))]
        return torch.cat(ys, dim=1)
    if kind == "forward":
        return _forward64(src["X"], *src["layer"], case["d_out"])
    if kind == "backward":
        Wp, C, piv, npiv = src["layer"]
        G = src["dY"].double()
        Gp = G[:, piv] + G[:, npiv] @ C.double()
        return {"dX": Gp @ Wp.double(), "dWp": Gp.t().contiguous() @ src["X"].double(),
                "dC": G[:, npiv].t().contiguous() @ src["Y"][:, piv].double()}
    if kind == "calibrate":
        S = torch.zeros((case["d_in"],) * 2, dtype=torch.float64, device=DEVICE)
        P = torch.zeros_like(S)
        for xo, xu in zip(src["Xo"], src["Xu"]):
            S += xu.double().t().contiguous() @ xu.double()
            P += xo.double().t().contiguous() @ xu.double()
        return {"S": S, "P": P}
    if kind == "reconstruct":
        xo, xu, W, V = src["Xo"].double(), src["Xu"].double(), src["W"], src["Vt"].t().contiguous()
        S = xu.t().contiguous() @ xu
        T = W @ (LAM * (xo.t().contiguous() @ xu) + (1 - LAM) * S)
        U_r = torch.linalg.solve(V.t() @ S @ V, (T @ V).t()).t()
        Q = torch.linalg.solve(U_r.t() @ U_r, U_r.t() @ (T + ALPHA * W))
        eye = torch.eye(case["d_in"], dtype=torch.float64, device=DEVICE)
        Vt_r = torch.linalg.solve(S + ALPHA * eye, Q.t()).t()
        return {"U_r": U_r.contiguous(), "Vt_r": Vt_r.contiguous()}
    W, U, r = src["W"], src["U"], case["r"]
    picked, diag = _pivoted_rows(W, r)
    piv = torch.sort(picked)[0]
    rest = torch.ones(W.shape[0], dtype=torch.bool, device=W.device)
    rest[piv] = False
    npiv = torch.nonzero(rest)[:, 0]
    # W' = U V: the non-pivot rows are U_np U_p^-1 times the pivot rows
    C = torch.linalg.solve(U[piv].t().contiguous(), U[npiv].t().contiguous()).t().contiguous()
    report = torch.tensor([float(diag[0]), float(diag[-1]), 0.0, 1.0], dtype=torch.float64)
    return {"piv": piv.to(torch.int32).cpu().numpy(), "npiv": npiv.to(torch.int32).cpu().numpy(), "Wp": W[piv],
            "C": C, "report": report.numpy()}
