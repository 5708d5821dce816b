"""The work a user has this library do, as cases that can be prepared, run and checked one by one.

A case is a dict of plain values.  `listed` are the fixed cases, `draw` makes
further ones of the same ranges, `prepare` makes what a caller has in hand
before the call (inputs, code, parity, buffers), `run` makes one pass through
the public calls of paper_1512_02673_amd.binding, and `exact` is the same
result in fp64 by plain torch, without the library's kernels.

Kinds:
  product  coded_matmul: draw the survivors, n worker products, decode (and the
           encode first when "encode" is set)
  gd       coded_gd_step: one iteration of coded gradient descent, two coded
           products with the residual and the update
  encode   coded_encode: the parity blocks of a matrix, once per matrix
  decode   coded_decode_batched: many survivor sets over one set of results
  shuffle  coded_shuffle_encode and coded_shuffle_decode of one planned iteration
  runtime  coded_simulate_runtimes: Monte-Carlo of the runtime model

The generator's parity rows come from "code_seed" and the survivors from
"draw_index", so the condition number of a case's decode system, which its
accuracy depends on, belongs to the case; the matrices come from the seed.
A shuffling plan, whose tables fix the sizes of the outputs, belongs to the
case too ("plan_seed").
"""
from __future__ import annotations

import math

import numpy as np
import torch

from paper_1512_02673_amd import binding as lib

SURVIVOR_SEED = 2
DT = {"f32": torch.float32, "bf16": torch.bfloat16}


def listed():
    return [
        # The smallest configured product, (4,2) on 2048 x 512, encoded and
        # multiplied per call: one short launch, so latency and host work count.
        _product("mds4x2_2048x512", 4, 2, 2048, 512, 1, encode=True),
        # The benchmark's default: a large matrix encoded once, a fresh vector
        # per call (serving one linear map).
        _product("gemv16x12_65536x8192", 16, 12, 65536, 8192, 1),
        # The matrix-vector experiment the method was published with: a (25,23)
        # code on 11500 x 5750, rows that are no multiple of 16 bytes.
        _product("gemv25x23_11500x5750", 25, 23, 11500, 5750, 1),
        # A batch of right-hand sides in fp32 (fp64 sums): several queries, or
        # the columns of a block method, per call.
        _product("gemm20x16_16384x4096x64", 20, 16, 16384, 4096, 64),
        # The same published code and matrix in bf16 with a small batch of
        # vectors, rows of 11500 bytes.
        _product("bf16_25x23_11500x5750x16", 25, 23, 11500, 5750, 16, dtype="bf16"),
        # The dense bf16 workload: encode, 64-column products and decode in
        # every call; the largest case.
        _product("dense32x24_131072x16384x64", 32, 24, 131072, 16384, 64, dtype="bf16", encode=True, code_seed=3),
        # Coded least squares at a published size, (10,8) codes on 10000 x 400:
        # short dependent launches, one iteration per call.
        {"name": "gd10x8_10000x400", "kind": "gd", "n": 10, "k": 8, "q": 10000, "r": 400, "planes": 2, "code_seed": 5},
        # Encoding a large matrix, done once per matrix before it is served.
        {"name": "encode16x12_65536x8192", "kind": "encode", "n": 16, "k": 12, "q": 65536, "r": 8192, "dtype": "f32",
         "planes": 2, "code_seed": 2},
        # The decode-heavy workload: many distinct survivor sets with at least
        # 8 missing blocks over one set of results.
        {"name": "decode64x48_16384x8_1000", "kind": "decode", "n": 64, "k": 48, "q": 16384, "s": 8, "batch": 1000,
         "min_parity": 8, "y": "f64", "code_seed": 4},
        # One coded shuffling iteration of the benchmark's size: 16 workers,
        # caches of a tenth of 10^6 rows of 1 KB.
        {"name": "shuffle16_1000000x256", "kind": "shuffle", "n": 16, "q": 1000000, "r": 256, "cache": 100000,
         "plan_seed": 8},
        # The runtime model at the published figure's (10,5), all three schemes.
        {"name": "runtime10x5_16M", "kind": "runtime", "n": 10, "k": 5, "count": 1 << 24, "repetition": True},
        # The runtime model of the largest configured code.
        {"name": "runtime64x48_1M", "kind": "runtime", "n": 64, "k": 48, "count": 1 << 20, "repetition": False},
    ]


def _product(name, n, k, q, r, s, dtype="f32", planes=2, encode=False, code_seed=2, draw_index=0):
    return {"name": name, "kind": "product", "n": n, "k": k, "q": q, "r": r, "s": s, "dtype": dtype, "planes": planes,
            "encode": encode, "code_seed": code_seed, "draw_index": draw_index}


CODES = [(3, 2), (4, 2), (5, 3), (10, 8), (16, 12), (20, 16), (25, 23), (32, 24), (64, 48)]


def _log(rng, lo, hi):
    """An integer of [lo, hi], uniform over its logarithm."""
    return min(hi, max(lo, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


def _matrix_size(rng, k, least, most, rmax=16384):
    """(q, r) of about 2^least .. 2^most elements; half of the row lengths are
    multiples of 64, the others whatever comes."""
    r = _log(rng, 64, rmax)
    if rng.random() < 0.5:
        r = max(64, r // 64 * 64)
    elements = 2.0 ** rng.uniform(least, most)
    return max(k, int(elements / r)), r


def draw(rng):
    kind = rng.choice(["vector", "vector", "columns", "bf16", "bf16", "gd", "encode", "decode", "shuffle", "runtime"])
    n, k = rng.choice(CODES)
    if kind in ("vector", "columns", "bf16"):
        dtype = "bf16" if kind == "bf16" else "f32"
        most = {"vector": 29, "columns": 26, "bf16": 29}[kind]
        q, r = _matrix_size(rng, k, 16, most)
        s = 1 if kind == "vector" or (kind == "bf16" and rng.random() < 0.25) else _log(rng, 2, 96)
        # one parity plane and the bfloat16 lo plane are fp32 options for vectors
        planes = rng.choice([2, 2, 1, lib.CODED_PLANES_LO_BF16]) if kind == "vector" else 2
        case = _product("", n, k, q, r, s, dtype, planes, rng.random() < 0.4, rng.randrange(1 << 16), 0)
        del case["name"]
        # bf16 results are documented up to decode systems of condition about
        # 8000; one draw in a thousand lies beyond
        while _condition(case) > 500:
            case["draw_index"] += 1
        return case
    if kind == "gd":
        n, k = rng.choice([(5, 3), (10, 8), (20, 16), (25, 23)])
        q, r = _matrix_size(rng, 64, 18, 28, 8192)
        if rng.random() < 0.5:
            q, r = max(q, 64), max(r, 64)
        return {"kind": "gd", "n": n, "k": k, "q": q, "r": r, "planes": 2, "code_seed": rng.randrange(1 << 16)}
    if kind == "encode":
        dtype = rng.choice(["f32", "f32", "bf16"])
        q, r = _matrix_size(rng, k, 16, 28)
        return {"kind": "encode", "n": n, "k": k, "q": q, "r": r, "dtype": dtype, "planes": 2,
                "code_seed": rng.randrange(1 << 16)}
    if kind == "decode":
        n, k = rng.choice([(16, 12), (20, 16), (32, 24), (64, 48), (96, 64), (128, 96)])
        s = rng.choice([1, 1, 2, 4, 8, rng.randrange(3, 65)])
        q = _log(rng, 1000, 65536)
        batch = _log(rng, 1, max(1, min(1000, (1 << 27) // (q * s))))
        return {"kind": "decode", "n": n, "k": k, "q": q, "s": s, "batch": batch, "min_parity": 0,
                "y": rng.choice(["f64", "f64", "f32"]), "code_seed": rng.randrange(1 << 16)}
    if kind == "shuffle":
        n = rng.choice([4, 8, 16, 16, 25, 32])
        q = _log(rng, 2000, 200000) // n * n
        cache = max(q // n, min(q, int(q * rng.uniform(0.05, 0.4))))
        r = _log(rng, 16, 2048)
        return {"kind": "shuffle", "n": n, "q": q, "r": r if rng.random() < 0.4 else max(16, r // 16 * 16),
                "cache": cache, "plan_seed": rng.randrange(1 << 16)}
    n = _log(rng, 3, 128)
    repetition = rng.random() < 0.5
    ks = [d for d in range(1, n + 1) if not repetition or n % d == 0]
    return {"kind": "runtime", "n": n, "k": rng.choice(ks), "count": _log(rng, 1 << 12, 1 << 22) * 4 // max(4, n // 8),
            "repetition": repetition}


# ------------------------------------------------------------------ codes


def _parity_rows(case, stream=0):
    """The parity rows P of the generator: i.i.d. N(0,1), rounded to the data's type."""
    g = np.random.default_rng([case["code_seed"], case["n"], case["k"], stream])
    p = torch.from_numpy(g.standard_normal((case["n"] - case["k"], case["k"])).astype(np.float32))
    if case.get("dtype") == "bf16":
        p = p.bfloat16().float()
    return p.double().numpy()


def _condition(case):
    """Condition number of the case's decode system (1 when no block is missing)."""
    n, k = case["n"], case["k"]
    surv, _ = lib.coded_draw_survivors(n, k, SURVIVOR_SEED, case["draw_index"])
    rows = [w - k for w in surv if w >= k]
    miss = sorted(set(range(k)) - {int(w) for w in surv})
    return float(np.linalg.cond(_parity_rows(case)[rows][:, miss])) if miss else 1.0


def _generator(seed, salt=0):
    return torch.Generator(device="cuda").manual_seed(seed * 1000003 + salt)


def _normal(shape, dtype, gen, std=1.0):
    """N(0, std^2) of `dtype` on the GPU, drawn in slabs so that no fp32 copy of a large bf16 matrix is held."""
    out = torch.empty(shape, dtype=dtype, device="cuda")
    rows = out.view(shape[0], -1)
    step = max(1, (1 << 26) // max(1, rows.shape[1]))
    for i in range(0, shape[0], step):
        part = rows[i:i + step]
        part.copy_(torch.randn(part.shape, dtype=torch.float32, device="cuda", generator=gen).mul_(std))
    return out


# ------------------------------------------------------------------ prepare and run


def prepare(case, seed):
    return {"product": _prepare_product, "gd": _prepare_gd, "encode": _prepare_encode, "decode": _prepare_decode,
            "shuffle": _prepare_shuffle, "runtime": _prepare_runtime}[case["kind"]](case, seed)


def run(state):
    return state["run"](state)


def _inputs(case, seed):
    dt = DT[case["dtype"]]
    A = _normal((case["q"], case["r"]), dt, _generator(seed, 1))
    X = _normal((case["r"], case["s"]), dt, _generator(seed, 2))
    return A, (X.view(-1) if case["s"] == 1 else X)


def _planes(code, parity, q, r, dtype):
    """The parity planes a caller looks at: hi and lo for fp32.  For bf16 the hi
    plane: lo is its rounding remainder, which no other implementation repeats
    value for value where hi rounds the other way; the results of the parity
    workers, returned beside it, depend on both."""
    if code.planes == lib.CODED_PLANES_LO_BF16:
        return list(lib.parity_planes(code, parity, q, r))
    return [parity[0]] if dtype == "bf16" else [parity[h] for h in range(code.planes)]


def _prepare_product(case, seed):
    n, k, q, r, s = (case[v] for v in ("n", "k", "q", "r", "s"))
    A, X = _inputs(case, seed)
    code = lib.Code.systematic(_parity_rows(case), case["planes"])
    parity = lib.alloc_parity(code, q, r, A.dtype)
    if not case["encode"]:
        lib.coded_encode(code, A, parity)
    ws = lib.matmul_workspace(code, A, X)
    y_dt, size = (torch.float64, 8) if case["dtype"] == "f32" else (torch.float32, 4)
    out = torch.empty((q, s) if s > 1 else (q,), dtype=torch.float32, device="cuda")
    st = {"run": _run_product, "code": code, "A": A, "X": X, "parity": parity, "ws": ws, "out": out,
          "info": torch.zeros(1, dtype=torch.int32, device="cuda"), "draw": case["draw_index"],
          "ready": not case["encode"]}
    # coded_matmul leaves every worker's result in the workspace
    qb = code.qb(q)
    st["result"] = {"out": out, "info": st["info"], "Y": ws[:n * qb * s * size].view(y_dt).view(n, qb, s)}
    if case["encode"]:
        st["result"]["parity"] = _planes(code, parity, q, r, case["dtype"])
    return st


def _run_product(st):
    lib.coded_matmul(st["code"], st["A"], st["parity"], st["X"], st["out"], st["ws"], st["info"], SURVIVOR_SEED,
                     st["draw"], parity_ready=st["ready"])
    return st["result"]


def _gd_step_size(q, r, std):
    """One over the largest eigenvalue of A^T A (its large-size value)."""
    return 1.0 / (std * std * (math.sqrt(q) + math.sqrt(r)) ** 2)


def _gd_inputs(case, seed):
    q, r = case["q"], case["r"]
    std = 1.0 / math.sqrt(r)
    A = _normal((q, r), torch.float32, _generator(seed, 1), std)
    w = _normal((r, 1), torch.float32, _generator(seed, 2))
    y = (A @ w).view(-1) + _normal((q, 1), torch.float32, _generator(seed, 3), 0.1).view(-1)
    x = _normal((r, 1), torch.float32, _generator(seed, 4), 0.5).view(-1)
    return A, y, x, _gd_step_size(q, r, std)


def _prepare_gd(case, seed):
    q, r = case["q"], case["r"]
    A, y, x, eta = _gd_inputs(case, seed)
    AT = torch.empty((r, q), dtype=torch.float32, device="cuda")
    lib.coded_transpose(A, AT)
    cA = lib.Code.systematic(_parity_rows(case, 0), case["planes"])
    cT = lib.Code.systematic(_parity_rows(case, 1), case["planes"])
    pA, pT = lib.alloc_parity(cA, q, r, torch.float32), lib.alloc_parity(cT, r, q, torch.float32)
    lib.coded_encode(cA, A, pA)
    lib.coded_encode(cT, AT, pT)
    return {"run": _run_gd, "cA": cA, "cT": cT, "A": A, "AT": AT, "pA": pA, "pT": pT, "y": y, "x": x, "eta": eta,
            "t": 0, "ws": torch.empty(lib.coded_gd_sizes(cA, cT, q, r), dtype=torch.uint8, device="cuda"),
            "info": torch.zeros(2, dtype=torch.int32, device="cuda")}


def _run_gd(st):
    lib.coded_gd_step(st["cA"], st["cT"], st["A"], st["pA"], st["AT"], st["pT"], st["y"], st["x"], st["eta"],
                      SURVIVOR_SEED, st["t"], st["ws"], st["info"])
    st["t"] += 1
    return {"x": st["x"], "info": st["info"]}


def _prepare_encode(case, seed):
    q, r = case["q"], case["r"]
    A = _normal((q, r), DT[case["dtype"]], _generator(seed, 1))
    code = lib.Code.systematic(_parity_rows(case), case["planes"])
    parity = lib.alloc_parity(code, q, r, A.dtype)
    return {"run": _run_encode, "code": code, "A": A, "parity": parity,
            "result": _planes(code, parity, q, r, case["dtype"])}


def _run_encode(st):
    lib.coded_encode(st["code"], st["A"], st["parity"])
    return st["result"]


def _decode_inputs(case, seed):
    """The k block products (fp64) and every worker's result."""
    k, q, s = case["k"], case["q"], case["s"]
    qb = -(-q // k)
    B = torch.zeros((k * qb, s), dtype=torch.float64, device="cuda")
    B[:q] = torch.randn((q, s), dtype=torch.float64, device="cuda", generator=_generator(seed, 1)) * 64.0
    B = B.view(k, qb * s)
    P = torch.from_numpy(_parity_rows(case)).cuda()
    Y = torch.cat([B, P @ B]).view(case["n"], qb, s)
    return B, (Y if case["y"] == "f64" else Y.float())


def _prepare_decode(case, seed):
    B, Y = _decode_inputs(case, seed)
    batch, q, s = case["batch"], case["q"], case["s"]
    sets, _ = lib.coded_draw_survivor_sets(case["n"], case["k"], seed, batch, min_parity=case["min_parity"])
    return {"run": _run_decode, "code": lib.Code.systematic(_parity_rows(case), 2), "Y": Y.contiguous(), "q": q,
            "sets": torch.from_numpy(sets).cuda(),
            "out": torch.zeros((batch, q, s) if s > 1 else (batch, q), dtype=torch.float32, device="cuda"),
            "info": torch.zeros(batch, dtype=torch.int32, device="cuda")}


def _run_decode(st):
    lib.coded_decode_batched(st["code"], st["sets"], st["Y"], st["q"], st["out"], st["info"])
    return {"out": st["out"], "info": st["info"]}


def _shuffle_plan(case):
    sh = lib.Shuffle(case["n"], case["q"], case["cache"], case["plan_seed"])
    sh.plan()
    tables = sh.tables()
    sh.close()
    return {name: torch.from_numpy(tables[name]).cuda() for name in ("enc_off", "enc_rows", "term_msg")}


def _prepare_shuffle(case, seed):
    q, r = case["q"], case["r"]
    A = _normal((q, r), torch.float32, _generator(seed, 1))
    tb = _shuffle_plan(case)
    return {"run": _run_shuffle, "A": A, "tb": tb,
            "M": torch.empty((tb["enc_off"].numel() - 1, r), dtype=torch.float32, device="cuda"),
            "out": torch.empty((tb["enc_rows"].numel(), r), dtype=torch.float32, device="cuda")}


def _run_shuffle(st):
    tb = st["tb"]
    lib.coded_shuffle_encode(st["A"], tb["enc_off"], tb["enc_rows"], st["M"])
    lib.coded_shuffle_decode(st["A"], st["M"], tb["enc_off"], tb["enc_rows"], tb["term_msg"], st["out"])
    return {"M": st["M"], "rows": st["out"]}


def _prepare_runtime(case, seed):
    new = lambda: torch.empty(case["count"], dtype=torch.float64, device="cuda")  # noqa: E731
    return {"run": _run_runtime, "n": case["n"], "k": case["k"], "seed": seed, "uncoded": new(),
            "repetition": new() if case["repetition"] else None, "mds": new()}


def _run_runtime(st):
    lib.coded_simulate_runtimes(st["n"], st["k"], st["seed"], 0, st["uncoded"], st["repetition"], st["mds"])
    return {name: st[name] for name in ("uncoded", "repetition", "mds")}


# ------------------------------------------------------------------ work, tolerance, exact


def work(case):
    kind, n, k = case["kind"], case["n"], case.get("k", 1)
    if kind == "runtime":
        count = case["count"]
        # about 20 operations for a worker's word, n log2 n comparisons to order them
        return {"bytes": 8.0 * count * (2 + case["repetition"]),
                "flops": count * n * (20.0 + max(1.0, math.log2(n)))}
    q = case["q"]
    qb = -(-q // k)
    if kind == "decode":
        size = 8.0 if case["y"] == "f64" else 4.0
        out = case["batch"] * q * case["s"]
        m = min(k, n - k) * 0.5
        return {"bytes": size * n * qb * case["s"] + 4.0 * out + 4.0 * case["batch"] * (k + 1),
                "flops": 2.0 * case["batch"] * m * k * qb * case["s"]}
    r = case["r"]
    if kind == "shuffle":
        # every worker lacks about (1 - cache / q) of its q / n rows; the multicast rows are at most as many
        rows = q * (1.0 - case["cache"] / q)
        return {"bytes": 4.0 * r * (q + 0.5 * rows + rows), "flops": 2.0 * r * rows}
    if kind == "gd":
        par = 2.0 * (n - k) * (qb * r + -(-r // k) * q)
        return {"bytes": 4.0 * (2.0 * q * r + par + 2.0 * q + 2.0 * r), "flops": 2.0 * (2.0 * q * r + par)}
    size = 4.0 if case["dtype"] == "f32" else 2.0
    element = 6.0 if case["planes"] == lib.CODED_PLANES_LO_BF16 else size * case["planes"]
    planes = 1 if case["planes"] == 1 else 2
    parity = (n - k) * qb * r
    enc = 2.0 * k * parity
    if kind == "encode":
        return {"bytes": size * q * r + element * parity, "flops": enc}
    s = case["s"]
    y = (8.0 if case["dtype"] == "f32" else 4.0) * n * qb * s
    return {"bytes": size * q * r + element * parity + size * r * s + y + 4.0 * q * s,
            "flops": 2.0 * s * (q * r + planes * parity) + (enc if case["encode"] else 0.0)}


def tolerance(case):
    if case["kind"] == "runtime":
        return {"rel": 1e-14}             # one fp64 logarithm: a few units in the last place
    if case["kind"] == "shuffle":
        return {"rel": 2e-7}              # a few fp32 sums in a fixed order
    if case.get("dtype") == "bf16":
        # fp32 sums, then a decode that multiplies their error by the condition
        # number (5e-6 off at 6, 1.1e-5 at 24); a stored bf16 value may round
        # the other way (half a percent of it)
        rel = 1e-4
        if case["kind"] == "product":
            rel = max(rel, 2e-6 * _condition(case))
        return {"rel": min(rel, 2e-2), "max": min(max(1e-2, 40 * rel), 0.5)}
    if case["kind"] == "gd":
        return {"rel": 1.5e-7}            # an fp32 residual between two fp64 products
    return {"rel": 1e-7}                  # fp64 sums, outputs rounded to fp32 (2.5e-8 off)


def exact(case, seed):
    return {"product": _exact_product, "gd": _exact_gd, "encode": _exact_encode, "decode": _exact_decode,
            "shuffle": _exact_shuffle, "runtime": _exact_runtime}[case["kind"]](case, seed)


def _times(A, X):
    """A X in fp64, a slab of rows at a time."""
    step = max(1, (1 << 27) // A.shape[1])
    Xd = X.double()
    return torch.cat([A[i:i + step].double() @ Xd for i in range(0, A.shape[0], step)])


def _exact_planes(case, A):
    """The parity planes: the fp64 sums rounded to the storage type, and the rounded remainder."""
    n, k, q, r = (case[v] for v in ("n", "k", "q", "r"))
    qb = -(-q // k)
    P = torch.from_numpy(_parity_rows(case)).cuda()
    low = torch.bfloat16 if case["planes"] == lib.CODED_PLANES_LO_BF16 else torch.float32
    planes = 1 if case["dtype"] == "bf16" or case["planes"] == 1 else 2
    out = [torch.empty((n - k, qb, r), dtype=torch.float64, device="cuda") for _ in range(planes)]
    step = max(1, (1 << 26) // (k * r))
    for t in range(0, qb, step):
        e = min(qb, t + step)
        part = torch.zeros((k, e - t, r), dtype=torch.float64, device="cuda")
        for j in range(k):
            rows = A[min(q, j * qb + t):min(q, j * qb + e)]
            part[j, :rows.shape[0]] = rows.double()
        total = (P @ part.view(k, -1)).view(n - k, e - t, r)
        hi = total.float().to(DT[case["dtype"]]).double()
        out[0][:, t:e] = hi
        if planes == 2:
            out[1][:, t:e] = (total - hi).float().to(low).double()
    return out


def _exact_product(case, seed):
    n, k, q, s = (case[v] for v in ("n", "k", "q", "s"))
    qb = -(-q // k)
    A, X = _inputs(case, seed)
    B = torch.zeros((k * qb, s), dtype=torch.float64, device="cuda")
    B[:q] = _times(A, X.view(-1, s))
    out = B[:q].clone() if s > 1 else B[:q, 0].clone()
    B = B.view(k, qb * s)
    P = torch.from_numpy(_parity_rows(case)).cuda()
    res = {"out": out, "info": None, "Y": torch.cat([B, P @ B]).view(n, qb, s)}
    if case["encode"]:
        res["parity"] = _exact_planes(case, A)
    return res


def _exact_gd(case, seed):
    A, y, x, eta = _gd_inputs(case, seed)
    z = _times(A, x.view(-1, 1)).view(-1) - y.double()
    step = max(1, (1 << 27) // A.shape[1])
    g = torch.zeros(case["r"], dtype=torch.float64, device="cuda")
    for i in range(0, A.shape[0], step):
        g += z[i:i + step] @ A[i:i + step].double()
    return {"x": x.double() - eta * g, "info": None}


def _exact_encode(case, seed):
    return _exact_planes(case, _normal((case["q"], case["r"]), DT[case["dtype"]], _generator(seed, 1)))


def _exact_decode(case, seed):
    B, _ = _decode_inputs(case, seed)
    q, s, batch = case["q"], case["s"], case["batch"]
    one = B.reshape(-1, s)[:q]
    one = one if s > 1 else one[:, 0]
    return {"out": one.expand(batch, *one.shape).contiguous(), "info": None}


def _exact_shuffle(case, seed):
    A = _normal((case["q"], case["r"]), torch.float32, _generator(seed, 1))
    tb = _shuffle_plan(case)
    M = torch.zeros((tb["enc_off"].numel() - 1, case["r"]), dtype=torch.float64, device="cuda")
    rows = tb["enc_rows"].long()
    M.index_add_(0, tb["term_msg"].long(), A[rows].double())
    return {"M": M, "rows": A[rows].double()}


def _signed(v):
    return v - (1 << 64) if v >= 1 << 63 else v


def _shr(x, n):
    return (x >> n) & ((1 << (64 - n)) - 1)


def _exact_runtime(case, seed):
    """SplitMix64 words (Steele, Lea, Flood 2014) of (draw, worker) in wrapping
    64-bit integers, ordered as the 53-bit uniforms they stand for."""
    n, k, count = case["n"], case["k"], case["count"]
    gamma, m1, m2 = (_signed(v) for v in (0x9E3779B97F4A7C15, 0xBF58476D1CE4E5B9, 0x94D049BB133111EB))
    got = {"uncoded": [], "repetition": [], "mds": []}
    step = max(1, (1 << 26) // n)
    for d in range(0, count, step):
        idx = torch.arange(d, min(count, d + step), dtype=torch.int64, device="cuda")
        word = _signed((4 << 56) & ((1 << 64) - 1)) + (idx[:, None] << 16) + torch.arange(n, device="cuda")[None, :]
        z = seed + (word + 1) * gamma
        z = (z ^ _shr(z, 30)) * m1
        z = (z ^ _shr(z, 27)) * m2
        z = z ^ _shr(z, 31)
        top = _shr(z, 11)

        def t0(v):
            return 1.0 - torch.log((v.double() + 0.5) * 2.0 ** -53)
        got["uncoded"].append(t0(top.amin(1)) / n)
        got["mds"].append(t0(torch.sort(top, dim=1, descending=True).values[:, k - 1]) / k)
        if case["repetition"]:
            got["repetition"].append(t0(top.view(-1, k, n // k).amax(2).amin(1)) / k)
    return {name: torch.cat(v) if v else None for name, v in got.items()}
