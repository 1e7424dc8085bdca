"""Workloads whose speed is measured, run through the library's public calls.

A case names a loop family and its sizes. `prepare` makes what a program has
in hand before the call (device arrays, loop handles, captured graphs),
`run` is one pass, `exact` gives the pass's results in float64 by plain
torch, `work` the bytes and operations a pass cannot do without.

All contexts enqueue on one stream, as one program would; each state has a
context of its own so that a cost model's weights belong to one state.
"""
import ctypes as C
import math

import numpy as np
import torch

from paper_2209_10643_amd import helpers as H
from paper_2209_10643_amd import upir as U

POLICY = {"auto": U.UPIR_SCHED_AUTO, "static": U.UPIR_SCHED_STATIC, "chunk": U.UPIR_SCHED_STATIC_CHUNK,
          "dynamic": U.UPIR_SCHED_DYNAMIC, "guided": U.UPIR_SCHED_GUIDED}
RED = {"sum": U.UPIR_RED_SUM, "max": U.UPIR_RED_MAX, "min": U.UPIR_RED_MIN}
DTYPE = {"f32": (U.UPIR_DT_F32, torch.float32), "f64": (U.UPIR_DT_F64, torch.float64),
         "i32": (U.UPIR_DT_I32, torch.int32), "i64": (U.UPIR_DT_I64, torch.int64)}
MATMUL = {"f32": U.UPIR_BODY_MATMUL_F32, "bf16": U.UPIR_BODY_MATMUL_BF16, "split": U.UPIR_BODY_MATMUL_SPLIT3}
A = 2.5  # the AXPY scalar


def listed():
    return [
        # the smallest call: the first size of the AXPY grid, with the sum of
        # y' that the one-loop workload reduces; latency and launches count
        {"name": "axpy_sum_10k", "family": "axpy", "n": 10240, "sched": "auto", "chunk": 0, "off": 0, "red": "sum"},
        # the largest size of the AXPY grid under the schedule its listing
        # names, schedule(static), teams and units chosen by the library
        {"name": "axpy_static_102m", "family": "axpy", "n": 102400000, "sched": "static", "chunk": 0, "off": 0,
         "red": "none"},
        # a standalone reduction of double-precision data, a ragged length
        {"name": "sum_f64_10m", "family": "sum", "n": 10000003, "dtype": "f64", "sched": "auto", "chunk": 0, "off": 0,
         "red": "sum"},
        # the headline workload: 100 sweeps with the largest update of every
        # sweep, captured once and replayed
        {"name": "jacobi_4096x100", "family": "jacobi", "rows": 4096, "cols": 4096, "sweeps": 100, "red": "max"},
        # one sweep over a grid whose rows are not a multiple of anything
        {"name": "jacobi_ragged", "family": "jacobi", "rows": 1501, "cols": 2003, "sweeps": 1, "red": "max"},
        # the three precisions of the matrix product: the size grid's largest
        # in float32, the 4096 cube in bfloat16, a ragged split product
        {"name": "matmul_f32_1024", "family": "matmul", "kind": "f32", "m": 1024, "n": 1024, "k": 1024},
        {"name": "matmul_bf16_4096", "family": "matmul", "kind": "bf16", "m": 4096, "n": 4096, "k": 4096},
        {"name": "matmul_split_ragged", "family": "matmul", "kind": "split", "m": 1000, "n": 1300, "k": 777},
        # the size grid's largest matrix-vector product
        {"name": "matvec_16384", "family": "matvec", "rows": 16384, "cols": 16384},
        # the size grid's largest 7 x 7 stencil
        {"name": "filter7_2048", "family": "filter7", "rows": 2048, "cols": 2048},
        # the batched workload: 2048 uneven tasks (AXPY, SUM, MATVEC) with
        # random depend edges in one captured launch
        {"name": "tasks_2048", "family": "tasks", "tasks": 2048, "lmax": 22, "degree": 2.0, "shared": False,
         "spec": 12345},
        # one training step of the schedule cost model at its batch size
        {"name": "model_step_256", "family": "model", "rows": 256, "train": True},
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    f = rng.choice(["axpy", "axpy", "sum", "sum", "jacobi", "jacobi", "matmul", "matmul", "matmul", "matvec", "matvec",
                    "filter7", "tasks", "model"])
    if f in ("axpy", "sum"):
        sched = rng.choice(["auto", "auto", "static", "chunk", "dynamic", "guided"])
        top = {"auto": 102400000, "static": 102400000}.get(sched, 5000000)
        c = {"family": f, "n": _log(rng, 1000, top), "sched": sched,
             "chunk": _log(rng, 16, 1024) if sched in ("chunk", "dynamic", "guided") else 0,
             "off": rng.choice([0, 0, 1, 2])}  # first element of the loop inside its array
        if f == "axpy":
            c["red"] = rng.choice(["none", "sum"]) if sched == "auto" else "none"
        else:
            c["dtype"] = rng.choice(["f32", "f64", "i32", "i64"])
            c["n"] = min(c["n"], 50000000)
            c["red"] = rng.choice(["sum", "sum", "max", "min"]) if c["dtype"] != "f32" or sched == "auto" else "max"
        return c
    if f == "jacobi":
        sweeps = rng.choice([1, 1, 10])
        return {"family": f, "rows": _log(rng, 60, 6000 if sweeps == 1 else 2000),
                "cols": _log(rng, 60, 6000 if sweeps == 1 else 2000), "sweeps": sweeps,
                "red": rng.choice(["none", "max", "max", "sum"])}
    if f == "matmul":
        # every size of a product has its own draw; half of them keep sizes
        # that are multiples of eight
        top = rng.choice([600, 2000])
        size = [_log(rng, 64, top) for _ in range(3)]
        if rng.random() < 0.5:
            size = [max(64, s // 8 * 8) for s in size]
        return {"family": f, "kind": rng.choice(["f32", "f32", "bf16", "split"]), "m": size[0], "n": size[1],
                "k": size[2]}
    if f == "matvec":
        rows = _log(rng, 16, 16384)
        return {"family": f, "rows": rows, "cols": _log(rng, 256, min(65536, 200000000 // rows))}
    if f == "filter7":
        return {"family": f, "rows": _log(rng, 64, 2048), "cols": _log(rng, 64, 2048)}
    if f == "tasks":
        return {"family": f, "tasks": _log(rng, 32, 1024), "lmax": rng.choice([14, 18, 20]),
                "degree": rng.choice([0.0, 1.0, 2.0, 4.0]), "shared": rng.random() < 0.5,
                "spec": rng.randrange(1 << 30)}
    train = rng.random() < 0.6
    return {"family": f, "rows": _log(rng, 16, 2048) if train else _log(rng, 16, 200000), "train": train}


class State:
    """A context, its handles and the arrays a pass works on."""

    _stream = None

    def __init__(self):
        if State._stream is None:
            State._stream = torch.cuda.Stream()
        self.ctx = H.Context(0, stream=State._stream)
        self.keep = []
        self.out = {}
        self.go = None

    def loop(self, kind, args, dims, sched=None, red=None):
        self.keep.append((args, sched, red))
        return self.ctx.loop(kind, args, dims, sched, red)

    def __del__(self):
        try:
            self.ctx.close()
        except Exception:
            pass


def _gen(seed):
    return torch.Generator(device="cuda").manual_seed(int(seed) * 7919 + 17)


def _pm1(g, *shape):
    return torch.rand(*shape, device="cuda", generator=g) * 2 - 1


def _sched(case):
    return None if case["sched"] == "auto" else H.make_sched(POLICY[case["sched"]], case["chunk"])


def _vectors(case, seed):
    g = _gen(seed)
    n = case["n"] + case["off"]
    if case["family"] == "axpy":
        return _pm1(g, n), _pm1(g, n)
    d = case["dtype"]
    if d[0] == "i":
        return (torch.randint(-1000, 1000, (n,), device="cuda", generator=g, dtype=DTYPE[d][1]),)
    return (torch.rand(n, device="cuda", generator=g, dtype=DTYPE[d][1]),)


def _grid(case, seed):
    u = torch.rand(case["rows"], case["cols"], device="cuda", generator=_gen(seed))
    u[0, :] = u[-1, :] = 0
    u[:, 0] = u[:, -1] = 0
    return u


def _operands(case, seed):
    g = _gen(seed)
    return (torch.randn(case["m"], case["k"], device="cuda", generator=g),
            torch.randn(case["k"], case["n"], device="cuda", generator=g))


def _matvec(case, seed):
    g = _gen(seed)
    return _pm1(g, case["rows"], case["cols"]), _pm1(g, case["cols"])


def _filter(case, seed):
    g = _gen(seed)
    return _pm1(g, case["rows"], case["cols"]), _pm1(g, 7, 7) * 0.25


# Task graph: kinds uniform over AXPY / SUM / MATVEC (rows x 256), lengths
# floor(2^U), U uniform in [8, lmax], an edge i < j with probability
# 2 degree / (tasks - 1). `shared`: a SUM whose first predecessor is an AXPY
# reduces that task's y instead of an array of its own.
def _graph(case):
    r = np.random.RandomState(case["spec"] % (1 << 32))
    n = case["tasks"]
    kinds = r.randint(0, 3, n)
    lens = np.floor(2.0 ** r.uniform(8, case["lmax"], n)).astype(np.int64)
    p = 2.0 * case["degree"] / max(1, n - 1)
    preds = [[int(i) for i in np.nonzero(r.random_sample(j) < p)[0]] for j in range(n)]
    tasks = []
    offs = {"x": 0, "y": 0, "A": 0, "v": 0, "w": 0}  # array starts, 256-byte aligned

    def take(role, count):
        at = offs[role]
        offs[role] += -(-count // 64) * 64
        return at

    for j in range(n):
        L = int(lens[j])
        if kinds[j] == 0:
            tasks.append({"kind": "axpy", "n": L, "x": take("x", L), "y": take("y", L)})
        elif kinds[j] == 1:
            src = preds[j][0] if case["shared"] and preds[j] and tasks[preds[j][0]]["kind"] == "axpy" else None
            if src is not None:
                tasks.append({"kind": "sum", "n": tasks[src]["n"], "of": src})
            else:
                tasks.append({"kind": "sum", "n": L, "x": take("x", L)})
        else:
            rows = max(1, L // 256)
            tasks.append({"kind": "matvec", "n": rows, "A": take("A", 256 * rows), "v": take("v", 256),
                          "w": take("w", rows)})
    return tasks, preds, offs


def _task_arrays(offs, seed):
    g = _gen(seed)
    a = {r: _pm1(g, max(64, offs[r])) for r in ("x", "y", "A", "v")}
    a["w"] = torch.zeros(max(64, offs["w"]), device="cuda")
    return a


def _model(case, seed):
    g = _gen(seed)
    w = []
    for fan_in, count in ((32, 64 * 32), (0, 64), (64, 64 * 64), (0, 64), (64, 64), (0, 1)):
        w.append(_pm1(g, count) * math.sqrt(6.0 / fan_in) if fan_in else _pm1(g, count) * 0.1)
    x = torch.rand(case["rows"], 32, device="cuda", generator=g)
    t = torch.rand(case["rows"], device="cuda", generator=g) * 8 + 2
    return torch.cat(w), x, t


def prepare(case, seed):
    s = State()
    f = case["family"]
    ctx = s.ctx
    if f == "axpy":
        x, y = _vectors(case, seed)
        r = torch.zeros(1, dtype=torch.float64, device="cuda")
        red = H.make_red(RED[case["red"]], r.data_ptr()) if case["red"] != "none" else None
        lp = s.loop(U.UPIR_BODY_AXPY, U.upir_axpy_args(A, 0, x.data_ptr(), y.data_ptr()),
                    [(case["off"], case["off"] + case["n"], 1)], _sched(case), red)
        s.keep.append((x, y, r))
        s.out = {"y": y, "s": r} if red is not None else {"y": y}
        s.go = lambda: ctx.launch(lp)
    elif f == "sum":
        (x,) = _vectors(case, seed)
        r = torch.zeros(1, dtype=torch.int64 if case["dtype"][0] == "i" else torch.float64, device="cuda")
        lp = s.loop(U.UPIR_BODY_SUM, U.upir_sum_args(x.data_ptr(), DTYPE[case["dtype"]][0], 0),
                    [(case["off"], case["off"] + case["n"], 1)], _sched(case),
                    H.make_red(RED[case["red"]], r.data_ptr()))
        s.keep.append((x, r))
        s.out = {"s": r}
        s.go = lambda: ctx.launch(lp)
    elif f == "jacobi":
        # sweep 1 reads the initial grid, later ones alternate between two
        # others, so a pass starts from the same grid every time
        u0 = _grid(case, seed)
        a, b = u0.clone(), u0.clone()
        k, W = case["sweeps"], case["cols"]
        res = torch.zeros(k, dtype=torch.float64, device="cuda")
        dims = [(1, case["rows"] - 1, 1), (1, W - 1, 1)]
        loops, src = [], u0
        for q in range(k):
            dst = a if q % 2 == 0 else b
            red = H.make_red(RED[case["red"]], res[q:].data_ptr(), async_=k > 1) if case["red"] != "none" else None
            loops.append(s.loop(U.UPIR_BODY_JACOBI5, U.upir_jacobi5_args(src.data_ptr(), dst.data_ptr(), W), dims,
                                None, red))
            src = dst
        s.keep.append((u0, a, b, res))
        s.out = {"u": src, "res": res} if case["red"] != "none" else {"u": src}
        if k == 1:
            s.go = lambda: ctx.launch(loops[0])
        else:
            torch.cuda.synchronize()
            ctx.launch(loops)
            ctx.sync()
            ctx.graph_begin()
            ctx.launch(loops)
            graph = ctx.graph_end()
            s.go = lambda: ctx.graph_launch(graph)
    elif f == "matmul":
        a, b = _operands(case, seed)
        m, n, k = case["m"], case["n"], case["k"]
        c = torch.zeros(m, n, device="cuda")
        lp = s.loop(MATMUL[case["kind"]],
                    U.upir_matmul_args(a.data_ptr(), b.data_ptr(), c.data_ptr(), k, k, n, n, None, 0),
                    [(0, m, 1), (0, n, 1)])
        s.keep.append((a, b, c))
        s.out = {"c": c}
        s.go = lambda: ctx.launch(lp)
    elif f == "matvec":
        a, x = _matvec(case, seed)
        y = torch.zeros(case["rows"], device="cuda")
        lp = s.loop(U.UPIR_BODY_MATVEC,
                    U.upir_matvec_args(a.data_ptr(), x.data_ptr(), y.data_ptr(), case["cols"], case["cols"]),
                    [(0, case["rows"], 1)])
        s.keep.append((a, x, y))
        s.out = {"y": y}
        s.go = lambda: ctx.launch(lp)
    elif f == "filter7":
        u, w = _filter(case, seed)
        v = torch.zeros_like(u)
        lp = s.loop(U.UPIR_BODY_FILTER7, U.upir_filter7_args(u.data_ptr(), v.data_ptr(), w.data_ptr(), case["cols"]),
                    [(3, case["rows"] - 3, 1), (3, case["cols"] - 3, 1)])
        s.keep.append((u, w, v))
        s.out = {"v": v}
        s.go = lambda: ctx.launch(lp)
    elif f == "tasks":
        tasks, preds, offs = _graph(case)
        arr = _task_arrays(offs, seed)
        sums = torch.zeros(len(tasks), dtype=torch.float64, device="cuda")
        tok = torch.zeros(len(tasks), dtype=torch.int64, device="cuda")
        at = {r: arr[r].data_ptr() for r in arr}
        torch.cuda.synchronize()
        for j, t in enumerate(tasks):
            if t["kind"] == "axpy":
                lp = s.loop(U.UPIR_BODY_AXPY, U.upir_axpy_args(A, 0, at["x"] + 4 * t["x"], at["y"] + 4 * t["y"]),
                            [(0, t["n"], 1)])
            elif t["kind"] == "sum":
                src = at["y"] + 4 * tasks[t["of"]]["y"] if "of" in t else at["x"] + 4 * t["x"]
                lp = s.loop(U.UPIR_BODY_SUM, U.upir_sum_args(src, U.UPIR_DT_F32, 0), [(0, t["n"], 1)], None,
                            H.make_red(U.UPIR_RED_SUM, sums.data_ptr() + 8 * j))
            else:
                lp = s.loop(U.UPIR_BODY_MATVEC,
                            U.upir_matvec_args(at["A"] + 4 * t["A"], at["v"] + 4 * t["v"], at["w"] + 4 * t["w"], 256,
                                               256), [(0, t["n"], 1)])
            deps = [(tok.data_ptr() + 8 * j, U.UPIR_DEP_OUT)]
            deps += [(tok.data_ptr() + 8 * i, U.UPIR_DEP_IN) for i in preds[j]]
            ctx.task(lp, deps)
        graph = ctx.taskwait_graph(U.UPIR_TASKWAIT_BATCHED)
        s.keep.append((arr, sums, tok))
        s.out = {"y": arr["y"], "sums": sums, "w": arr["w"]}
        s.go = lambda: ctx.graph_launch(graph)
    else:
        w, x, t = _model(case, seed)
        U.upir_model_init(ctx.h, 1)
        host = w.cpu().numpy()
        U.upir_model_set_params(ctx.h, host.ctypes.data_as(C.POINTER(C.c_float)))
        rows, h = case["rows"], ctx.h
        xp, tp = x.data_ptr(), t.data_ptr()
        if case["train"]:
            grad = torch.zeros(U.UPIR_MLP_PARAMS, device="cuda")
            gp = grad.data_ptr()
            s.keep.append((x, t, grad))
            s.out = {"grad": grad}
            s.go = lambda: U.upir_model_step(h, xp, tp, rows, 1e-3, 1, gp, None)
        else:
            y = torch.zeros(rows, device="cuda")
            yp = y.data_ptr()
            s.keep.append((x, y))
            s.out = {"y": y}
            s.go = lambda: U.upir_model_forward(h, xp, rows, yp)
    return s


def run(state):
    state.go()
    return state.out


def work(case):
    f = case["family"]
    if f == "axpy":
        return {"bytes": 12 * case["n"], "flops": (3 if case["red"] != "none" else 2) * case["n"]}
    if f == "sum":
        return {"bytes": (4 if case["dtype"][1:] == "32" else 8) * case["n"], "flops": case["n"]}
    if f == "jacobi":
        r, c = case["rows"], case["cols"]
        return {"bytes": case["sweeps"] * (4 * r * c + 4 * (r - 2) * (c - 2)),
                "flops": case["sweeps"] * (r - 2) * (c - 2) * (4 if case["red"] == "none" else 7)}
    if f == "matmul":
        m, n, k = case["m"], case["n"], case["k"]
        return {"bytes": 4 * (m * k + k * n + m * n), "flops": 2 * m * n * k * (3 if case["kind"] == "split" else 1)}
    if f == "matvec":
        return {"bytes": 4 * (case["rows"] * (case["cols"] + 1) + case["cols"]), "flops": 2 * case["rows"] * case["cols"]}
    if f == "filter7":
        r, c = case["rows"], case["cols"]
        return {"bytes": 4 * r * c + 4 * (r - 6) * (c - 6), "flops": 98 * (r - 6) * (c - 6)}
    if f == "tasks":
        b = fl = 0
        for t in _graph(case)[0]:
            b += {"axpy": 12, "sum": 4, "matvec": 1028}[t["kind"]] * t["n"] + (1024 if t["kind"] == "matvec" else 8)
            fl += {"axpy": 2, "sum": 1, "matvec": 512}[t["kind"]] * t["n"]
        return {"bytes": b, "flops": fl}
    n, params = case["rows"], U.UPIR_MLP_PARAMS
    if case["train"]:  # forward, two products backward, Adam on the weights
        return {"bytes": 4 * n * 33 + 4 * params * 7, "flops": 6 * n * 6208}
    return {"bytes": 4 * n * 33 + 4 * params, "flops": 2 * n * 6208}


def _reduce(v, op):
    return v.sum() if op == "sum" else v.max().clamp(min=0) if op == "max" else v.min().clamp(max=0)


def exact(case, seed):
    f = case["family"]
    if f == "axpy":
        x, y = (v.double() for v in _vectors(case, seed))
        lo = case["off"]
        y[lo:] += A * x[lo:]
        if case["red"] == "none":
            return {"y": y}
        return {"y": y, "s": y[lo:].float().double().sum().reshape(1)}
    if f == "sum":
        (x,) = _vectors(case, seed)
        if case["dtype"][0] == "i":
            return None
        return {"s": _reduce(x[case["off"]:].double(), case["red"]).reshape(1)}
    if f == "jacobi":
        u = _grid(case, seed).double()
        res = []
        for _ in range(case["sweeps"]):
            v = u.clone()
            v[1:-1, 1:-1] = ((u[:-2, 1:-1] + u[2:, 1:-1]) + (u[1:-1, :-2] + u[1:-1, 2:])) * 0.25
            if case["red"] != "none":
                res.append(_reduce((v - u)[1:-1, 1:-1].abs(), case["red"]))
            u = v
        return {"u": u, "res": torch.stack(res)} if res else {"u": u}
    if f == "matmul":
        a, b = _operands(case, seed)
        if case["kind"] == "f32":
            return {"c": a.double() @ b.double()}
        ah, bh = a.bfloat16(), b.bfloat16()
        c = ah.double() @ bh.double()
        if case["kind"] == "split":
            al, bl = (a - ah.float()).bfloat16().double(), (b - bh.float()).bfloat16().double()
            c += al @ bh.double() + ah.double() @ bl
        return {"c": c}
    if f == "matvec":
        a, x = _matvec(case, seed)
        return {"y": a.double() @ x.double()}
    if f == "filter7":
        u, w = (v.double() for v in _filter(case, seed))
        r, c = case["rows"] - 6, case["cols"] - 6
        v = torch.zeros_like(u)
        for m in range(7):
            for n in range(7):
                v[3:-3, 3:-3] += w[m, n] * u[m:m + r, n:n + c]
        return {"v": v}
    if f == "tasks":
        tasks, _, offs = _graph(case)
        arr = _task_arrays(offs, seed)
        sums = torch.zeros(len(tasks), dtype=torch.float64, device="cuda")
        w = arr["w"].double()
        y, y32 = arr["y"].double(), arr["y"]
        for j, t in enumerate(tasks):
            n = t["n"]
            if t["kind"] == "axpy":
                y[t["y"]:t["y"] + n] += A * arr["x"][t["x"]:t["x"] + n].double()
                y32[t["y"]:t["y"] + n] = y[t["y"]:t["y"] + n].float()
            elif t["kind"] == "sum":
                v = y32[tasks[t["of"]]["y"]:][:n] if "of" in t else arr["x"][t["x"]:][:n]
                sums[j] = v.double().sum()
            else:
                a = arr["A"][t["A"]:t["A"] + 256 * n].view(n, 256).double()
                w[t["w"]:t["w"] + n] = (a * arr["v"][t["v"]:t["v"] + 256].double()).sum(1)
        return {"y": y, "sums": sums, "w": w}
    p, x, t = (v.double() for v in _model(case, seed))
    w1, b1, w2, b2, w3, b3 = torch.split(p, [64 * 32, 64, 64 * 64, 64, 64, 1])
    w1, w2 = w1.view(64, 32), w2.view(64, 64)
    z1 = x @ w1.t().contiguous() + b1
    h1 = z1.clamp(min=0)
    z2 = h1 @ w2.t().contiguous() + b2
    h2 = z2.clamp(min=0)
    y = h2 @ w3 + b3
    if not case["train"]:
        return {"y": y}
    dy = 2.0 * (y - t) / case["rows"]
    d2 = dy[:, None] * w3 * (z2 > 0)
    d1 = (d2 @ w2) * (z1 > 0)
    g = [d1.t().contiguous() @ x, d1.sum(0), d2.t().contiguous() @ h1, d2.sum(0), h2.t().contiguous() @ dy, dy.sum()]
    return {"grad": torch.cat([v.reshape(-1) for v in g])}
