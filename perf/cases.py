"""The calls whose speed matters, as a program that serves CTR models makes them.

Each case is one pass through a public entry point: a whole lookup step
(``FusedLookup``: plan, then lookup), the FM term over a pooled block, a step
that starts from the data loader's host arrays, or the interaction head.  The
listed cases are the repository's workloads from its smallest (eight one-hot
fields, 256 samples) to its largest (100 fields of up to 10 M rows, 65,536
samples); ``draw`` gives more of the same ranges.
"""
from __future__ import annotations

import math
from typing import Dict, List, Optional

import numpy as np
import torch

from paper_2606_21101_amd import dpi
from paper_2606_21101_amd.lookup import FusedLookup

_TORCH = {"f32": torch.float32, "f16": torch.float16}
_DPI = {"f32": dpi.DPI_F32, "f16": dpi.DPI_F16}
_X = {"i64": (torch.int64, dpi.DPI_X_I64), "i32": (torch.int32, dpi.DPI_X_I32), "f32": (torch.float32, dpi.DPI_X_F32)}
_POOL = {"sum": lambda t: 0, "mean": lambda t: 1, "alternate": lambda t: t % 2}


def _lookup(name: Optional[str] = None, **kw) -> dict:
    """A lookup case.  bags: "onehot" (no offsets), "poisson" (mean bag_mean,
    clipped to [bag_lo, bag_hi]), "lognormal" (median bag_mean, sigma
    bag_sigma), "mixed" (the first third of the fields one-hot, the others
    Poisson with a mean of their own up to bag_mean, one bag in twenty empty).
    Row counts are log-uniform in [rows_lo, rows_hi]; ids follow a bounded Zipf
    law of exponent zipf over the rows (0: uniform)."""
    case = {"kind": "lookup", "fields": 26, "batch": 4096, "rows_lo": 1000, "rows_hi": 1000000, "dims": "16",
            "table": "f32", "out": "f32", "bags": "onehot", "bag_mean": 1.0, "bag_sigma": 0.0, "bag_lo": 0,
            "bag_hi": 256, "zipf": 1.05, "pooling": "sum", "shape_seed": 1}
    case.update(kw)
    if name is not None:
        case["name"] = name
    return case


def listed() -> List[dict]:
    hetero = dict(fields=39, rows_lo=10, rows_hi=10_000_000, dims="8,16,32,64", bags="mixed", bag_mean=40.0, zipf=1.2)
    return [
        # the smallest batch the repository measures: a ranking call over a few fields, all launch and latency
        _lookup("tiny_onehot", fields=8, batch=256, rows_lo=1000, rows_hi=1000, zipf=0.0),
        # an ordinary one-hot CTR batch (26 fields, dim 16)
        _lookup("ctr_onehot", rows_lo=10),
        # the largest one-hot batch, with rows that are no power of two (dim 60)
        _lookup("onehot_dim60", batch=65536, rows_lo=500_000, rows_hi=500_000, dims="60"),
        # one sample over one-hot and multi-hot fields of several dims: an online request
        _lookup("request_b1", batch=1, **hetero),
        # the same model on a small serving batch: its lookup is the step's only launch
        _lookup("serve_b512", batch=512, **hetero),
        # ... and on a batch that needs a planning launch of its own
        _lookup("serve_b4096", batch=4096, **hetero),
        # multi-hot binary16 fields of one dim, the workload the paper's multi-hot discussion describes
        _lookup("multihot", batch=16384, rows_hi=5_000_000, dims="64", table="f16", out="f16", bags="poisson",
                bag_mean=10.0, bag_lo=1, bag_hi=64),
        # the largest workload: 100 fields, 59 GB of tables, sum and mean pooling
        _lookup("large", fields=100, batch=65536, rows_lo=100_000, rows_hi=10_000_000, dims="128", table="f16",
                out="f16", bags="lognormal", bag_mean=20.0, bag_sigma=0.8, zipf=1.1, pooling="alternate"),
        # rows that are no multiple of 16 bytes (dims 10, 18, 6, 50 of a hand-tuned model) beside one that is,
        # at an odd batch size
        _lookup("odd_dims", fields=24, batch=3001, dims="10,18,6,36,50", bags="poisson", bag_mean=6.0,
                pooling="alternate"),
        # DeepFM's second-order term over the multi-hot workload's pooled block
        {"name": "fm_multihot", "kind": "fm", "batch": 16384, "fields": 26, "dim": 64, "table": "f16"},
        # a serving step from the data loader's host CSR: one copy, the conversion, plan and lookup
        dict(_lookup("host_csr_b512", batch=512, **hetero), kind="stage", x="i64"),
        # the DCN interaction head (cross network and MLP) over 26 fields of dim 16, both modules overlapped
        {"name": "dcn_head", "kind": "dcn", "batch": 4096, "dim": 416, "cross": 3, "mlp": "1024,512,256"},
    ]


def _log_int(rng, lo: float, hi: float) -> int:
    return int(min(hi, max(lo, math.exp(rng.uniform(math.log(lo), math.log(hi + 1))))))


def draw(rng) -> dict:
    """One more case of the listed ones' ranges."""
    kind = rng.choice(["onehot", "multihot", "multihot", "mixed", "mixed", "odd", "fm", "stage", "dcn"])
    seed = rng.randrange(1, 1 << 30)
    table = rng.choice(["f32", "f16"])
    out = table if rng.random() < 0.7 else "f32"
    pooling = rng.choice(["sum", "mean", "alternate"])
    fields = rng.randint(4, 60)
    rows_lo = _log_int(rng, 10, 100_000)
    common = dict(fields=fields, rows_lo=rows_lo, rows_hi=_log_int(rng, rows_lo, 2_000_000), table=table, out=out,
                  zipf=rng.choice([0.0, 1.05, 1.1, 1.2]), pooling=pooling, shape_seed=seed)
    if kind == "onehot":
        return _lookup(batch=_log_int(rng, 64, 65536), dims=str(rng.choice([8, 16, 32, 60, 64, 100, 128])), **common)
    if kind == "multihot":
        return _lookup(batch=_log_int(rng, 2000, 40000), dims=str(rng.choice([16, 32, 64, 128])), bag_lo=0,
                       bags=rng.choice(["poisson", "lognormal"]), bag_mean=rng.uniform(3, 24), bag_sigma=0.8, **common)
    if kind == "mixed":
        return _lookup(batch=_log_int(rng, 1, 6000), dims="8,16,32,64", bags="mixed", bag_mean=rng.uniform(5, 40),
                       **common)
    if kind == "odd":
        dims = ",".join(str(2 * rng.randint(1, 40)) for _ in range(rng.randint(1, 5)))
        return _lookup(batch=_log_int(rng, 16, 8000), dims=dims, bags="poisson", bag_mean=rng.uniform(1, 12), **common)
    if kind == "fm":
        return {"kind": "fm", "batch": _log_int(rng, 100, 65536), "fields": rng.randint(4, 100),
                "dim": rng.choice([8, 10, 16, 32, 60, 64, 128]), "table": table}
    if kind == "stage":
        return dict(_lookup(batch=_log_int(rng, 1, 4096), dims="8,16,32,64", bags="mixed", bag_mean=rng.uniform(5, 40),
                            **common), kind="stage", x=rng.choice(["i64", "i32", "f32"]))
    return {"kind": "dcn", "batch": _log_int(rng, 64, 16384), "dim": rng.choice([128, 208, 390, 416, 624]),
            "cross": rng.randint(1, 4), "mlp": ",".join(str(rng.choice([64, 128, 200, 256, 512, 1024]))
                                                        for _ in range(rng.randint(1, 3)))}


# ---------------------------------------------------------------------------
# shapes that follow from a case alone
# ---------------------------------------------------------------------------
def _dims(case) -> List[int]:
    d = [int(x) for x in case["dims"].split(",")]
    return [d[t % len(d)] for t in range(case["fields"])]


def _rows(case) -> List[int]:
    rng = np.random.default_rng(case["shape_seed"])
    u = rng.uniform(math.log(case["rows_lo"]), math.log(case["rows_hi"]), case["fields"])
    return [int(n) for n in np.clip(np.exp(u).astype(np.int64), case["rows_lo"], case["rows_hi"])]


def _means(case) -> List[float]:
    """Expected ids per bag of every field (of the law before clipping)."""
    T = case["fields"]
    if case["bags"] == "onehot":
        return [1.0] * T
    if case["bags"] == "mixed":
        rng = np.random.default_rng(case["shape_seed"] + 1)
        lam = rng.uniform(1.0, case["bag_mean"], T)
        return [1.0 if t < T // 3 else float(lam[t]) for t in range(T)]
    if case["bags"] == "lognormal":
        return [case["bag_mean"] * math.exp(case["bag_sigma"] ** 2 / 2) - 0.5] * T
    return [case["bag_mean"]] * T


def _distinct(n: int, draws: float, s: float) -> float:
    """Expected number of distinct rows among `draws` draws from the id law over n rows."""
    if s == 0.0:
        return n * -math.expm1(draws * math.log1p(-1.0 / n)) if n > 1 else 1.0
    edges = np.unique(np.round(np.geomspace(1, n + 1, 4000)).astype(np.int64))   # rank ranges [edges[i], edges[i+1])
    if len(edges) < 2:
        return 1.0
    width = np.diff(edges).astype(np.float64)
    mid = np.sqrt(edges[:-1] * np.maximum(edges[1:] - 1.0, edges[:-1]))
    w = mid ** -s
    p = np.minimum(w / np.sum(w * width), 1.0 - 1e-12)
    return float(np.sum(width * -np.expm1(draws * np.log1p(-p))))


# ---------------------------------------------------------------------------
# what a program holds before the call
# ---------------------------------------------------------------------------
def _gen(seed: int) -> torch.Generator:
    gen = torch.Generator(device="cuda")
    gen.manual_seed(seed)
    return gen


def _lengths(case, seed: int) -> torch.Tensor:
    T, B = case["fields"], case["batch"]
    # host arrays hold the same number of ids for every seed (their conversion is an output): one draw of lengths,
    # its samples rotated by the seed
    gen = _gen(case["shape_seed"] if case["kind"] == "stage" else seed + 1)
    lam = torch.tensor(_means(case), device="cuda")[:, None].expand(T, B).contiguous()
    if case["bags"] == "lognormal":
        z = torch.randn((T, B), generator=gen, device="cuda")
        n = torch.floor(case["bag_mean"] * torch.exp(case["bag_sigma"] * z))
    else:
        n = torch.poisson(lam, generator=gen)
    if case["bags"] == "mixed":
        n = torch.clamp(n, min=1)
        n[torch.rand((T, B), generator=gen, device="cuda") < 0.05] = 0
        n[: T // 3] = 1
    n = torch.clamp(n, case["bag_lo"], case["bag_hi"]).to(torch.int64)
    return torch.roll(n, seed % B, 1) if case["kind"] == "stage" else n


def _ids(n: int, count: int, s: float, gen) -> torch.Tensor:
    u = torch.rand(count, generator=gen, device="cuda", dtype=torch.float64)
    if s == 0.0:
        return torch.clamp((u * n).to(torch.int32), max=n - 1)
    cdf = torch.arange(1, n + 1, device="cuda", dtype=torch.float64).pow_(-s).cumsum_(0)
    return torch.clamp(torch.searchsorted(cdf, u.mul_(cdf[-1]), right=True), max=n - 1).to(torch.int32)


def _batch(case, seed: int) -> Dict[str, object]:
    """Tables N(0, 0.01) and one batch (int32 field-major CSR ids)."""
    T, B = case["fields"], case["batch"]
    gen = _gen(seed)
    tables = []
    for n, d in zip(_rows(case), _dims(case)):
        t = torch.empty((n, d), dtype=_TORCH[case["table"]], device="cuda")
        tables.append(t.normal_(0.0, 0.01, generator=gen))
    offsets = None
    counts = [B] * T
    if case["bags"] != "onehot":
        offsets = torch.zeros((T, B + 1), dtype=torch.int32, device="cuda")
        offsets[:, 1:] = torch.cumsum(_lengths(case, seed), 1)
        counts = [int(c) for c in offsets[:, -1].cpu()]
    ids = torch.cat([_ids(n, c, case["zipf"], gen) for n, c in zip(_rows(case), counts)])
    return {"tables": tables, "ids": ids, "offsets": offsets, "counts": counts,
            "pooling": [_POOL[case["pooling"]](t) for t in range(T)]}


def _dcn_weights(case, gen):
    d, mlp = case["dim"], [int(x) for x in case["mlp"].split(",")]

    def w(o, i):
        return torch.empty((o, i), device="cuda").normal_(0.0, 1.0 / math.sqrt(i), generator=gen)

    def b(o):
        return torch.empty(o, device="cuda").normal_(0.0, 0.1, generator=gen)

    cw, cb = [w(d, d) for _ in range(case["cross"])], [b(d) for _ in range(case["cross"])]
    mw = [w(o, i) for o, i in zip(mlp, [d] + mlp[:-1])]
    mb = [b(o) for o in mlp]
    x0 = torch.empty((case["batch"], d), device="cuda").normal_(0.0, 1.0, generator=gen)
    return cw, cb, mw, mb, x0


def prepare(case, seed):
    gen = _gen(seed)
    B = case["batch"]
    if case["kind"] == "fm":
        block = torch.empty((B, case["fields"] * case["dim"]), dtype=_TORCH[case["table"]], device="cuda")
        return {"case": case, "block": block.normal_(0.0, 0.03, generator=gen),
                "y": torch.empty(B, dtype=torch.float32, device="cuda")}
    if case["kind"] == "dcn":
        cw, cb, mw, mb, x0 = _dcn_weights(case, gen)
        return {"case": case, "x0": x0, "head": dpi.DcnHead(B, case["dim"], cw, cb, mw, mb),
                "cross": torch.empty_like(x0), "mlp": torch.empty((B, mb[-1].numel()), device="cuda"),
                "streams": (torch.cuda.Stream(), torch.cuda.Stream())}
    data = _batch(case, seed)
    fl = FusedLookup(data["tables"], data["pooling"], _TORCH[case["out"]])
    out = torch.empty((B, fl.total_dim), dtype=_TORCH[case["out"]], device="cuda")
    state = {"case": case, "fl": fl, "ids": data["ids"], "offsets": data["offsets"], "out": out}
    if case["kind"] == "stage":
        packed = torch.cat([data["offsets"].reshape(-1), data["ids"]]).to(_X[case["x"]][0])
        host = torch.empty(packed.shape, dtype=packed.dtype, pin_memory=True)
        state["packed"] = host.copy_(packed)
        state["staging"] = torch.empty_like(packed)
        state["ids"], state["offsets"] = torch.empty_like(data["ids"]), torch.empty_like(data["offsets"])
    return state


def run(state):
    case = state["case"]
    if case["kind"] == "fm":
        dpi.dpi_fm_second_order(state["block"], _DPI[case["table"]], case["batch"], case["fields"], case["dim"],
                                case["fields"] * case["dim"], state["y"])
        return state["y"]
    if case["kind"] == "dcn":
        s = state["streams"]
        state["head"].forward(state["x0"], state["cross"], state["mlp"], dpi.DPI_SCHED_BREADTH_FIRST, s[0], s[1])
        return {"cross": state["cross"], "mlp": state["mlp"]}
    if case["kind"] == "stage":
        dpi.dpi_stage_csr(state["packed"], _X[case["x"]][1], case["fields"], case["batch"], state["ids"].numel(),
                          state["staging"], state["offsets"], state["ids"])
        out = state["fl"](state["ids"], state["offsets"], case["batch"], out=state["out"])
        return {"ids": state["ids"], "offsets": state["offsets"], "out": out}
    return state["fl"](state["ids"], state["offsets"], case["batch"], out=state["out"])


# ---------------------------------------------------------------------------
# what a pass cannot do without, and how exact it is
# ---------------------------------------------------------------------------
def work(case):
    B = case["batch"]
    size = {"f32": 4, "f16": 2, "i64": 8, "i32": 4}
    if case["kind"] == "fm":
        n = B * case["fields"] * case["dim"]
        return {"bytes": n * size[case["table"]] + 4 * B, "flops": 3 * n}
    if case["kind"] == "dcn":
        d, mlp = case["dim"], [int(x) for x in case["mlp"].split(",")]
        cells = case["cross"] * d * d + sum(o * i for o, i in zip(mlp, [d] + mlp[:-1]))
        return {"bytes": 4 * (cells + B * (2 * d + mlp[-1])), "flops": 2 * B * cells}
    total, adds = 0.0, 0.0
    for n, d, m in zip(_rows(case), _dims(case), _means(case)):
        ids = m * B
        total += _distinct(n, ids, case["zipf"]) * d * size[case["table"]] + 4 * ids + B * d * size[case["out"]]
        adds += ids * d
        if case["bags"] != "onehot":
            total += 4 * (B + 1)
        if case["kind"] == "stage":   # the host's offsets and ids, read from host memory
            total += size[case["x"]] * (ids + B + 1)
    return {"bytes": total, "flops": adds}


def tolerance(case):
    if case["kind"] == "fm":
        return {"rel": 6e-7}
    if case["kind"] == "dcn":
        return {"rel": 3e-6}
    if case["bags"] == "onehot" and case["table"] == case["out"]:
        return "exact"
    return {"rel": 1e-3 if case["out"] == "f16" else 5e-7}


def exact(case, seed):
    B = case["batch"]
    if case["kind"] == "fm":
        e = prepare(case, seed)["block"].view(B, case["fields"], case["dim"])
        y = [0.5 * (c.double().sum(1).square() - c.double().square().sum(1)).sum(1) for c in e.split(4096)]
        return torch.cat(y)
    if case["kind"] == "dcn":
        cw, cb, mw, mb, x0 = _dcn_weights(case, _gen(seed))
        x = x0 = x0.double()
        h = x0
        for w, b in zip(cw, cb):
            x = x0 * (x @ w.double().t() + b.double()) + x
        for w, b in zip(mw, mb):
            h = torch.relu(h @ w.double().t() + b.double())
        return {"cross": x, "mlp": h}
    data = _batch(case, seed)
    out = torch.zeros((B, sum(_dims(case))), dtype=torch.float64, device="cuda")
    base, col = 0, 0
    for t, (table, count) in enumerate(zip(data["tables"], data["counts"])):
        d = table.shape[1]
        ids = data["ids"][base: base + count].long()
        if data["offsets"] is None:
            out[:, col: col + d] = table[ids].double()
        else:
            lens = torch.diff(data["offsets"][t]).long()
            bag = torch.repeat_interleave(torch.arange(B, device="cuda"), lens)
            pooled = torch.zeros((B, d), dtype=torch.float64, device="cuda").index_add_(0, bag, table[ids].double())
            if data["pooling"][t]:
                pooled /= torch.clamp(lens, min=1)[:, None].double()
            out[:, col: col + d] = pooled
        base, col = base + count, col + d
    if case["kind"] == "stage":
        return {"ids": data["ids"], "offsets": data["offsets"], "out": out}
    return out
