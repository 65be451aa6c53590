"""The work a user of the library has it do, as cases that can be timed.

A case is a dict of plain values; its "kind" names the part of the protocol:

  server   the server's product  Yhat = W Xhat mod p
  keygen   Preprocess: P^T and Q of one matrix
  step     one whole query batch on the one-call path:
           encode -> server_eval -> decode_verify
  client   the client's side of one query batch with prepared masks (the boost
           and standard modes): client_prepare, encode_masked and, on the
           server's response, decode_verify_masked
  layer    one decoder layer of the stack (seven projections, four inputs):
           preparation, then the online part
  batch    Protocol Batch-vMVMD: the server's projection and the client's checks

Every case goes through the package's public functions.  "graph": the calls of
the pass are captured once into a HIP graph that a pass replays, as a serving
program does (and as the repository's benchmark does) where launches of a few
microseconds follow one another; without it the functions are called.

Every value is an integer mod p, so every result is exact.
"""
import math

import torch

import paper_2609_10264_amd as mvk
from paper_2609_10264_amd import stack

TY, ELL = 31, 2  # weight and repetitions of the challenge (t_y and ell of the paper, Sec. 7.1)


# ---------------------------------------------------------------------------
# The cases
# ---------------------------------------------------------------------------
def listed():
    return [
        # One token through an attention projection: a single-query product, the
        # smallest server call of the configured workloads.
        dict(name="server_4096_b1", kind="server", m=4096, n=4096, B=1, packed=True, field="m31"),
        # An MLP up-projection with 16 query columns in flight.
        dict(name="server_11008x4096_b16", kind="server", m=11008, n=4096, B=16, packed=True, field="m31"),
        # The largest batched call: a 28672 x 8192 layer with 64 columns.
        dict(name="server_28672x8192_b64", kind="server", m=28672, n=8192, B=64, packed=True, field="m31"),
        # A matrix of odd sizes as the caller has it (row-major, not packed), over the
        # paper's field: pruned or unpadded projections.
        dict(name="server_ragged_rowmajor_b12", kind="server", m=5003, n=3001, B=12, packed=False, field="babybear"),
        # Preprocess of an MLP projection (what loading a model costs, per matrix).
        dict(name="keygen_11008x4096_r3", kind="keygen", m=11008, n=4096, r=3, field="m31"),
        # Preprocess at a size of the paper's own evaluation (rate 1/8, BabyBear).
        dict(name="keygen_8192_r8", kind="keygen", m=8192, n=8192, r=8, field="babybear"),
        # The smallest configuration, end to end: launches and latency only.
        dict(name="step_256_b1", kind="step", m=256, n=256, B=1, r=2, tx=8, field="m31", graph=True),
        # One query through an attention projection, end to end.
        dict(name="step_4096_b1", kind="step", m=4096, n=4096, B=1, r=3, tx=64, field="m31", graph=True),
        # The largest size of the paper's evaluation, end to end (block length 131072).
        dict(name="step_16384_b1", kind="step", m=16384, n=16384, B=1, r=8, tx=154, field="babybear", graph=False),
        # The client's side of the largest batched layer.
        dict(name="client_28672x8192_b64", kind="client", m=28672, n=8192, B=64, r=4, tx=128, field="m31",
             graph=False),
        # A decoder layer with 8 query columns (one of the 32 layers of the stack).
        dict(name="layer_b8", kind="layer", B=8, r=3, tx=64, field="m31", graph=True),
        # Batch verification of four claims of 4096 x 4096.
        dict(name="batch_4x4096", kind="batch", m=4096, n=4096, B=4, r=3, field="m31", graph=False),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _size(rng, lo, hi):
    """A length: half of them whole 64s (model dimensions), half of them any number."""
    v = _log(rng, lo, hi)
    return max(64, v // 64 * 64) if rng.random() < 0.5 else v


def draw(rng):
    kind = rng.choice(["server", "server", "server", "keygen", "step", "step", "client", "layer", "batch"])
    field = rng.choice(["m31", "m31", "babybear"])
    if kind == "server":
        while True:
            m, n, B = _size(rng, 256, 28672), _size(rng, 256, 16384), _log(rng, 1, 64)
            if m * n <= 28672 * 8192:
                return dict(kind=kind, m=m, n=n, B=B, packed=rng.random() < 0.7, field=field)
    if kind == "keygen":
        while True:
            m, n, r = _size(rng, 256, 16384), _size(rng, 256, 16384), rng.choice([2, 3, 4, 8])
            if r * m * n <= 8 * 8192 * 8192:
                return dict(kind=kind, m=m, n=n, r=r, field=field)
    if kind in ("step", "client"):
        while True:
            m, n, r = _size(rng, 256, 28672), _size(rng, 256, 16384), rng.choice([2, 3, 4, 8])
            B, tx = _log(rng, 1, 32), rng.choice([8, 64, 128, 154])
            if r * m * n <= 4 * 28672 * 8192 and r * max(m, n) <= 131072:
                return dict(kind=kind, m=m, n=n, B=B, r=r, tx=tx, field=field, graph=m * n * B <= 2**26)
    if kind == "layer":
        return dict(kind=kind, B=_log(rng, 1, 16), r=3, tx=rng.choice([32, 64]), field="m31", graph=True)
    while True:
        m, n, B = _size(rng, 256, 8192), _size(rng, 256, 8192), rng.randint(2, 6)
        if m * n * B * B <= 16 * 4096 * 4096 and 2 * B * n <= 65536:
            return dict(kind=kind, m=m, n=n, B=B, r=rng.choice([2, 3]), field=field, graph=False)


# ---------------------------------------------------------------------------
# Inputs, from the seed alone
# ---------------------------------------------------------------------------
def _p(case):
    return mvk.FIELDS[case["field"]]


class _Draw:
    def __init__(self, seed, p):
        self.g = torch.Generator(device="cuda")
        self.g.manual_seed(int(seed))
        self.p = p

    def weights(self, m, n):
        return torch.randint(-127, 128, (m, n), dtype=torch.int8, device="cuda", generator=self.g)

    def field(self, shape, lo=0):
        return torch.randint(lo, self.p, shape, dtype=torch.int32, device="cuda", generator=self.g)

    def code(self, k, r):
        pi = [torch.randperm(k * r, dtype=torch.int32, device="cuda", generator=self.g) for _ in range(2)]
        return mvk.Code(k, r, pi[0], pi[1], self.field((k * r,), 1), self.field((k * r,), 1), p=self.p)

    def sparse(self, count, N, t):
        """`count` vectors of exactly t nonzeros: distinct positions in random order, nonzero values."""
        t = min(t, N)
        pos = torch.rand((count, N), device="cuda", generator=self.g).topk(t, dim=1).indices.to(torch.int32)
        return pos.contiguous(), self.field((count, t), 1)


def _inputs(case, seed):
    """Every random draw of a case, in one order for prepare() and exact()."""
    d = _Draw(seed, _p(case))
    kind = case["kind"]
    s = {}
    if kind == "layer":
        B, r, tx = case["B"], case["r"], case["tx"]
        s["cx"], s["cy"] = stack.codes_for(lambda which, k: d.code(k, r))
        s["W"] = {nm: d.weights(m, n) for nm, m, n, _ in stack.PROJECTIONS}
        s["X"] = {g: d.field((B, stack.input_width(g))) for g in stack.INPUTS}
        s["ex"] = {g: d.sparse(B, stack.input_width(g) * r, tx) for g in stack.INPUTS}
        s["ey"] = {nm: d.sparse(ELL, m * r, TY) for nm, m, _, _ in stack.PROJECTIONS}
        return s
    m, n = case["m"], case["n"]
    if kind == "batch":
        B, r = case["B"], case["r"]
        s["cx"], s["cy"], s["c2"] = d.code(n, 2), d.code(m, r), d.code(B * n, 2)
        s["W"] = [d.weights(m, n) for _ in range(B)]
        s["X"] = d.field((B, n))
        s["e"], s["e2"] = d.sparse(ELL, m * r, TY), d.sparse(ELL, 2 * B * n, TY)
        return s
    s["W"] = d.weights(m, n)
    if kind == "server":
        s["X"] = d.field((case["B"], n))  # a masked query is uniform in the field
        return s
    s["cx"], s["cy"] = d.code(n, case["r"]), d.code(m, case["r"])
    if kind == "keygen":
        return s
    s["X"] = d.field((case["B"], n))
    s["ex"], s["ey"] = d.sparse(case["B"], n * case["r"], case["tx"]), d.sparse(ELL, m * case["r"], TY)
    return s


def _empty(*shape):
    return torch.empty(shape, dtype=torch.int32, device="cuda")


_side = None


def _captured(fn):
    """fn's calls as a HIP graph, captured on one side stream (the library's
    workspace is per stream: the call before the capture sizes it)."""
    global _side
    if _side is None:
        _side = torch.cuda.Stream()
    _side.wait_stream(torch.cuda.current_stream())
    with torch.cuda.stream(_side):
        fn()
    torch.cuda.synchronize()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g, stream=_side):
        out = fn()
    return g, out


def prepare(case, seed):
    s = _inputs(case, seed)
    kind, p = case["kind"], _p(case)
    if kind == "server":
        W = mvk.pack_weights(s["W"]) if case["packed"] else s["W"]
        out = _empty(case["B"], case["m"])
        call = lambda: mvk.server_eval(W, s["X"], out=out, p=p)  # noqa: E731
    elif kind == "keygen":
        key = mvk.Key.allocate(case["m"], case["n"], s["cx"], s["cy"])

        def call():
            mvk.keygen(key, s["W"])
            return {"PT": key.PT, "Q": key.Q}
    elif kind == "step":
        B, m, n = case["B"], case["m"], case["n"]
        key = mvk.keygen(mvk.Key.allocate(m, n, s["cx"], s["cy"]), s["W"])
        W = mvk.pack_weights(s["W"])
        xh, yh, y, vl, vr, acc = _empty(B, n), _empty(B, m), _empty(B, m), _empty(ELL, B), _empty(ELL, B), _empty(B)

        def call():
            mvk.encode(key, s["X"], *s["ex"], out=xh)
            mvk.server_eval(W, xh, out=yh, p=p)
            mvk.decode_verify(key, xh, yh, *s["ex"], *s["ey"], Y=y, vL=vl, vR=vr, accept=acc)
            return {"Xhat": xh, "Yhat": yh, "Y": y, "vL": vl, "vR": vr, "accept": acc}
    elif kind == "client":
        B, m, n = case["B"], case["m"], case["n"]
        key = mvk.keygen(mvk.Key.allocate(m, n, s["cx"], s["cy"]), s["W"])
        prep = mvk.Prepared(key, B, ELL)
        xh, y, vl, vr, acc = _empty(B, n), _empty(B, m), _empty(ELL, B), _empty(ELL, B), _empty(B)
        # the server's response, which the client's program has received
        yh = mvk.server_eval(mvk.pack_weights(s["W"]), mvk.encode(key, s["X"], *s["ex"]), p=p)
        del s["W"]

        def call():
            mvk.client_prepare(key, *s["ex"], *s["ey"], out=prep)
            mvk.encode_masked(key, s["X"], prep, out=xh)
            mvk.decode_verify_masked(key, xh, yh, prep, Y=y, vL=vl, vR=vr, accept=acc)
            return {"Mx": prep.Mx, "My": prep.My, "R": prep.R, "U": prep.U, "Xhat": xh, "Y": y, "vL": vl, "vR": vr,
                    "accept": acc}
    elif kind == "layer":
        layer = stack.build_layer(s["W"], s["cx"], s["cy"])
        preps = {}
        stack.prepare_layer(layer, s["ex"], s["ey"], None, out=preps)

        def call():
            stack.prepare_layer(layer, s["ex"], s["ey"], None, out=preps)
            res = stack.run_layer_prepared(layer, s["X"], preps)
            return {nm: {"Y": r[0], "accept": r[1], "Yhat": r[3], "vL": r[4], "vR": r[5]} for nm, r in res.items()}
    else:  # batch
        B, m, n = case["B"], case["m"], case["n"]
        Qs = [mvk.keygen(mvk.Key.allocate(m, n, s["cx"], s["cy"]), W).Q for W in s["W"]]
        QtT, Qaux = mvk.batch_preprocess(Qs, s["c2"])
        del Qs
        Y = torch.cat([mvk.server_eval(W, s["X"][b:b + 1].contiguous(), p=p) for b, W in enumerate(s["W"])])
        del s["W"]
        ut = _empty(ELL, B * n)
        vl, vr, sl, sr, acc = _empty(ELL, B), _empty(ELL, B), _empty(ELL, ELL), _empty(ELL, ELL), _empty(B)

        def call():
            mvk.batch_project(QtT, n, *s["e"], out=ut, p=p)
            mvk.batch_verify(s["cy"], s["c2"], Qaux, s["X"], Y, *s["e"], ut, *s["e2"], vL=vl, vR=vr, sL=sl, sR=sr,
                             accept=acc)
            return {"Ut": ut, "vL": vl, "vR": vr, "sL": sl, "sR": sr, "accept": acc}
    state = {"call": call, "inputs": s}
    if case.get("graph"):
        state["graph"], state["out"] = _captured(call)
    return state


def run(state):
    if "graph" in state:
        state["graph"].replay()
        return state["out"]
    return state["call"]()


# ---------------------------------------------------------------------------
# What a pass cannot do without
# ---------------------------------------------------------------------------
def _server_work(m, n, B):
    # an int8 weight times a 31-bit element is four int8 products
    return m * n + 4 * B * (m + n), 8 * m * n * B


def _code_bytes(k, r):
    return 16 * k * r  # two permutations, two diagonals


def _prep_work(m, n, B, r, tx):
    # noise in, input and output masks out, t_x rows of P^T a column; R and U, t_y rows of Q a repetition
    by = 8 * B * tx + 4 * B * (n + m) + 4 * B * tx * m + 8 * ELL * TY + 4 * ELL * (m + n) + 4 * ELL * TY * n
    return by + _code_bytes(n, r) + _code_bytes(m, r), 2 * B * tx * m + 2 * ELL * TY * n + 4 * r * (B * n + ELL * m)


def _check_work(m, n, B):
    # Xhat, Yhat, My, R, U in, Y out
    return 4 * B * (n + 3 * m) + 4 * ELL * (m + n), 2 * ELL * B * (m + n) + B * m


def work(case):
    kind = case["kind"]
    if kind == "layer":
        B, r, tx = case["B"], case["r"], case["tx"]
        by = fl = 0
        for nm, m, n, _ in stack.PROJECTIONS:
            for b, f in (_server_work(m, n, B), _check_work(m, n, B)):
                by, fl = by + b, fl + f
            by += 4 * B * m * (tx + 1) + 4 * ELL * TY * n + 4 * ELL * (m + n)
            fl += 2 * B * tx * m + 2 * ELL * TY * n + 4 * r * ELL * m
        for g in stack.INPUTS:
            n = stack.input_width(g)
            by, fl = by + 4 * B * 3 * n + 8 * B * tx, fl + 4 * r * B * n
        return {"bytes": by + 2 * (_code_bytes(4096, r) + _code_bytes(11008, r)), "flops": fl}
    m, n, B = case["m"], case["n"], case.get("B", 1)
    if kind == "server":
        by, fl = _server_work(m, n, B)
    elif kind == "keygen":
        r = case["r"]
        by = m * n + 8 * r * m * n + _code_bytes(n, r) + _code_bytes(m, r)
        fl = 8 * r * m * n  # two sums and two scalings of every entry of P^T and of Q
    elif kind in ("step", "client"):
        by, fl = _prep_work(m, n, B, case["r"], case["tx"])
        cb, cf = _check_work(m, n, B)
        by, fl = by + cb + 4 * B * n, fl + cf
        if kind == "step":
            sb, sf = _server_work(m, n, B)
            by, fl = by - 8 * B * m - 8 * B * n + sb, fl + sf  # no masks are written: they stay inside the calls
    else:
        r = case["r"]
        by = 4 * ELL * TY * B * n + 4 * ELL * B * n + 4 * B * (m + n) + 4 * ELL * ELL * TY * TY
        by += _code_bytes(m, r) + _code_bytes(B * n, 2)
        fl = 2 * ELL * TY * B * n + 4 * ELL * (r * m + 2 * B * n) + 2 * ELL * B * (2 * n + m)
    return {"bytes": by, "flops": fl}


def tolerance(case):
    return "exact"


# ---------------------------------------------------------------------------
# The same values from the definitions, in 64-bit torch
# ---------------------------------------------------------------------------
def _matmul(W, X, p):
    """X W^T mod p for int8 W (m x n) and X (B x n) in [0, p): the two 16-bit
    halves of X in float64, whose sums stay below 2^53."""
    Wt = W.double().t()
    lo, hi = (X.long() & 0xFFFF).double() @ Wt, (X.long() >> 16).double() @ Wt
    return (lo.long() % p + (hi.long() % p) * 65536) % p


def _dot(a, b, p):
    """sum over the last axis of a b mod p."""
    return ((a.long() * b.long()) % p).sum(-1) % p


def _syndrome(code, idx, val):
    """G e for each sparse vector (App. B): suffix sum, scale, scatter, suffix sum, scale, scatter, fold."""
    p, out = code.p, []
    for i, v in zip(idx.long(), val.long()):
        x = torch.zeros(code.N, dtype=torch.int64, device=idx.device)
        x[i] = v
        for pi, d in ((code.pi2, code.v2), (code.pi1, code.v1)):
            x = (x.flip(0).cumsum(0).flip(0) % p) * d.long() % p
            x = torch.empty_like(x).index_copy_(0, pi.long(), x)
        out.append(x.view(code.k, code.r).sum(1) % p)
    return torch.stack(out)


def _encode_cols(code, W):
    """G^T W for W (k x count) as int32 N x count, some columns at a time."""
    p = code.p
    out = torch.empty((code.N, W.shape[1]), dtype=torch.int32, device=W.device)
    step = max(1, 2**26 // code.N)
    for c in range(0, W.shape[1], step):
        x = W[:, c:c + step].long()[code.pi1.long() // code.r]
        x = (x * code.v1.long()[:, None] % p).cumsum(0) % p
        x = (x[code.pi2.long()] * code.v2.long()[:, None] % p).cumsum(0) % p
        out[:, c:c + step] = x.int()
    return out


def exact(case, seed):
    s = _inputs(case, seed)
    kind, p = case["kind"], _p(case)
    if kind == "server":
        return _matmul(s["W"], s["X"], p).int()
    if kind == "keygen":
        return {"PT": _encode_cols(s["cx"], s["W"].t()), "Q": _encode_cols(s["cy"], s["W"])}

    def checks(W, X, Xhat, R):
        Yhat = _matmul(W, Xhat, p)
        v = _dot(R[:, None, :], Yhat[None], p).int()  # an honest response: both sides are the same number
        return {"Y": _matmul(W, X, p).int(), "accept": torch.ones_like(v[0]), "Yhat": Yhat.int(), "vL": v, "vR": v}

    if kind == "layer":
        xh = {g: (s["X"][g].long() + _syndrome(s["cx"][stack.input_width(g)], *s["ex"][g])) % p for g in stack.INPUTS}
        return {nm: checks(s["W"][nm], s["X"][g], xh[g], _syndrome(s["cy"][m], *s["ey"][nm]))
                for nm, m, _, g in stack.PROJECTIONS}
    if kind == "batch":
        R = _syndrome(s["cy"], *s["e"])
        ut = torch.cat([_matmul(W.t(), R, p) for W in s["W"]], dim=1)
        Y = torch.cat([_matmul(W, s["X"][b:b + 1], p) for b, W in enumerate(s["W"])])
        v = _dot(R[:, None, :], Y[None], p).int()
        sv = _dot(ut[:, None, :], _syndrome(s["c2"], *s["e2"])[None], p).int()
        return {"Ut": ut.int(), "vL": v, "vR": v, "sL": sv, "sR": sv, "accept": torch.ones_like(v[0])}
    Mx, R = _syndrome(s["cx"], *s["ex"]), _syndrome(s["cy"], *s["ey"])
    Xhat = (s["X"].long() + Mx) % p
    out = checks(s["W"], s["X"], Xhat, R)
    out["Xhat"] = Xhat.int()
    if kind == "client":
        del out["Yhat"]
        out.update(Mx=Mx.int(), My=_matmul(s["W"], Mx, p).int(), R=R.int(), U=_matmul(s["W"].t(), R, p).int())
    return out
