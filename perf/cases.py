"""Performance cases of the mapping-search library: what its users have it do, over the real range.

A case is a dict of plain values.  `prepare` turns it and a seed into the structures a program holds
before the call (the seed moves the accelerator: buffer capacity, DRAM energy, for sweeps every
accelerator; for cost windows also where the window starts), `run` is one call through the public
entry points, `exact` restates the model in plain torch for the outputs that are computed numbers.
"""
import math
import random

import numpy as np

import paper_2604_03446_amd as M

KEYS = {"energy": M.OBJ_ENERGY, "latency": M.OBJ_LATENCY, "latency_then_energy": M.OBJ_LATENCY_THEN_ENERGY, "edp": M.OBJ_EDP}
DATAFLOW_ROWS = 37500       # (order, levels, recompute, fused) rows that denote a dataflow
KEPT_ROWS = 270             # rows the offline stage keeps


# ---- the cases ---------------------------------------------------------------------------------

def _attention(N, d, H, mode=0, c_softmax=10):
    return {"batch": H, "I": N, "K": d, "L": N, "J": d, "mode": mode, "c_softmax": c_softmax, "attention": True}


def _chain(I, K, L, J, mode=0):
    return {"batch": 1, "I": I, "K": K, "L": L, "J": J, "mode": mode, "c_softmax": 0, "attention": False}


def _accel(pe_rows, pe_cols, gb_kib, rf, whole=True, dram_bw=64.0, gb_bw=256.0, n_arrays=1):
    return {"pe_rows": pe_rows, "pe_cols": pe_cols, "gb_kib": gb_kib, "rf": rf, "whole": whole,
            "dram_bw": dram_bw, "gb_bw": gb_bw, "n_arrays": n_arrays}


def listed():
    return [
        # One mapping for one layer, as a compiler asks for it: the smallest problem, latency counts.
        {"name": "search_tiny", "kind": "search", "exhaustive": False, "keys": "energy", **_attention(64, 32, 1), **_accel(8, 8, 16, 64)},
        # The same for a prefill layer, latency first.
        {"name": "search_prefill", "kind": "search", "exhaustive": False, "keys": "latency_then_energy",
         **_attention(2048, 128, 32), **_accel(32, 32, 1024, 512)},
        # A sequence length that is no power of two, every divisor a tile size, an array and bandwidths
        # that are no powers of two, fractional energies; both metrics at once.
        {"name": "search_ragged", "kind": "search", "exhaustive": False, "keys": "energy+latency",
         **_attention(3000, 80, 24, mode=1), **_accel(24, 9, 300, 200, whole=False, dram_bw=60.0, gb_bw=200.0, n_arrays=3)},
        # Hardware design exploration: 64 accelerators x 8 attention shapes x 2 objectives in one call.
        {"name": "sweep_hardware", "kind": "sweep", "exhaustive": False, "n_hw": 64, "Ns": "512,1024,4096,16384", "ds": "64,128",
         "H": 16, "keys": "energy,latency"},
        # Exhaustive search of the long-context configuration (the library's headline).
        {"name": "exhaustive_long", "kind": "search", "exhaustive": True, "keys": "energy",
         **_attention(8192, 128, 32, mode=1), **_accel(128, 128, 8192, 1024)},
        # Exhaustive search for both metrics in one pass.
        {"name": "exhaustive_bert", "kind": "search", "exhaustive": True, "keys": "energy+latency",
         **_attention(512, 64, 12), **_accel(16, 16, 256, 256)},
        # Exhaustive search of two back-to-back GEMMs (a feed-forward layer) on a multi-array accelerator
        # whose DRAM bandwidth is no power of two.
        {"name": "exhaustive_ffn", "kind": "search", "exhaustive": True, "keys": "energy",
         **_chain(2048, 768, 3072, 768), **_accel(32, 32, 1024, 512, dram_bw=60.0, n_arrays=4)},
        # The energy-latency front a designer looks at.
        {"name": "front_energy_latency", "kind": "pareto", "exhaustive": False,
         **_attention(1024, 96, 16, mode=1), **_accel(16, 64, 512, 128, whole=False, dram_bw=16.0, gb_bw=128.0)},
        # How much buffer buys how much DRAM traffic.
        {"name": "front_buffer_dram", "kind": "front", "exhaustive": False, **_attention(512, 64, 12), **_accel(16, 16, 256, 256)},
        # Cost records of a long run of candidates into device memory (a learned cost model's training set).
        {"name": "records_device", "kind": "records", "n": 1 << 25, "host": False, **_attention(512, 64, 12), **_accel(16, 16, 256, 256)},
        # A short window of cost records into host memory, sixteen of them decoded: looking at the neighbours of a mapping.
        {"name": "records_host", "kind": "records", "n": 1 << 14, "host": True, **_attention(512, 64, 12), **_accel(16, 16, 256, 256)},
        # The search that allocates nothing and does not wait, from a serving loop.
        {"name": "noalloc_bert", "kind": "noalloc", "exhaustive": False, "keys": "energy", **_attention(512, 64, 12), **_accel(16, 16, 256, 256)},
    ]


def _divisors(x, mode):
    out = []
    for a in range(1, math.isqrt(x) + 1):
        if x % a == 0:
            out += [a, x // a]
    return sorted(v for v in set(out) if mode or v & (v - 1) == 0)


def _tilings(c):
    n = 1
    for q in "IKLJ":
        n *= len(_divisors(c[q], c["mode"]))
    return n


def _log_int(rng, lo, hi):
    return min(hi, max(lo, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


def _draw_shape(rng, most_tilings):
    while True:
        mode = rng.randrange(2)
        grain = rng.choice([1, 2, 8, 12, 60, 128])
        extent = lambda lo, hi: max(1, _log_int(rng, lo, hi) // grain) * grain  # noqa: E731
        if rng.random() < 0.7:
            c = _attention(extent(64, 16384), rng.choice([32, 40, 48, 64, 72, 75, 80, 96, 112, 128]), _log_int(rng, 1, 64), mode)
        else:
            c = _chain(extent(64, 12544), extent(16, 1024), extent(64, 4096), extent(16, 1024), mode)
        # the library keeps every count below 2^53
        if 36 <= _tilings(c) <= most_tilings and c["batch"] * c["I"] * c["K"] * c["L"] * c["J"] * 52 < 1 << 53:
            return c


def _draw_accel(rng):
    if rng.random() < 0.6:
        pe = 8 << rng.randrange(5)
        rows, cols = pe, pe
    else:
        rows, cols = rng.randrange(4, 129), rng.randrange(4, 129)
    return _accel(rows, cols, _log_int(rng, 16, 16384), 2 * _log_int(rng, 32, 1024), rng.random() < 0.5, rng.choice([16.0, 60.0, 64.0, 128.0]),
                  rng.choice([128.0, 200.0, 256.0]), rng.choice([1, 1, 2, 3, 4]))


def draw(rng):
    kind = rng.choice(["search", "search", "search", "sweep", "exhaustive", "exhaustive", "pareto", "front", "records", "records", "noalloc"])
    if kind == "sweep":
        Ns = rng.sample([256, 384, 512, 768, 1000, 1024, 1536, 2048, 3072, 4096, 8192, 16384], rng.randrange(1, 5))
        ds = rng.sample([48, 64, 80, 96, 128], rng.randrange(1, 3))
        return {"kind": "sweep", "exhaustive": False, "n_hw": _log_int(rng, 4, 64), "Ns": ",".join(map(str, Ns)),
                "ds": ",".join(map(str, ds)), "H": rng.choice([8, 12, 16, 32]), "keys": rng.choice(["energy", "latency", "energy,latency", "edp"])}
    if kind in ("search", "exhaustive"):
        keys = rng.choice(["energy", "latency", "latency_then_energy", "edp", "energy+latency"])
        return {"kind": "search", "exhaustive": kind == "exhaustive", "keys": keys,
                **_draw_shape(rng, 6000 if kind == "exhaustive" else 102400), **_draw_accel(rng)}
    if kind == "records":
        host = rng.random() < 0.5
        return {"kind": "records", "n": _log_int(rng, 1 << 8, 1 << 16) if host else _log_int(rng, 1 << 12, 1 << 25), "host": host,
                **_draw_shape(rng, 12544), **_draw_accel(rng)}
    shape = _draw_shape(rng, 12544)
    while kind == "noalloc" and not shape["attention"]:
        shape = _draw_shape(rng, 12544)
    c = {"kind": kind, "exhaustive": False, **shape, **_draw_accel(rng)}
    if kind == "noalloc":
        c["keys"] = rng.choice(["energy", "latency", "latency_then_energy", "edp"])
    return c


# ---- preparing and running ---------------------------------------------------------------------

def _problem(c):
    if c["attention"]:
        return dict(B=1, H=c["batch"], N=c["I"], d=c["K"], word_bytes=2, tiling_mode=c["mode"], c_softmax=c["c_softmax"])
    return dict(batch=c["batch"], I=c["I"], K=c["K"], L=c["L"], J=c["J"], word_bytes=2, tiling_mode=c["mode"], c_softmax=c["c_softmax"])


def _hardware(c, rng):
    """The case's accelerator with the seed's buffer capacity and DRAM energy."""
    e_dram = float(rng.randrange(100, 301)) if c["whole"] else rng.uniform(100.0, 300.0)
    gb = max(8, int(c["gb_kib"] * rng.uniform(0.75, 1.25))) * 1024
    return dict(pe_rows=c["pe_rows"], pe_cols=c["pe_cols"], n_arrays=c["n_arrays"], rf_bytes=c["rf"], gb_bytes=gb, e_dram=e_dram,
                e_gb=6.0, e_rf=1.0, e_mac=1.0, dram_bw=c["dram_bw"], gb_bw=c["gb_bw"])


def _sweep(c, rng):
    points = []
    hws = [dict(pe_rows=(pe := 8 << rng.randrange(5)), pe_cols=pe, n_arrays=1, rf_bytes=64 << rng.randrange(6), gb_bytes=(64 * 1024) << rng.randrange(9),
                e_dram=rng.uniform(100.0, 300.0), e_gb=6.0, e_rf=1.0, e_mac=1.0, dram_bw=64.0, gb_bw=256.0) for _ in range(c["n_hw"])]
    for N in map(int, c["Ns"].split(",")):
        for d in map(int, c["ds"].split(",")):
            w = M.workload(dict(B=1, H=c["H"], N=N, d=d, word_bytes=2, tiling_mode=0, c_softmax=10))
            points += [(w, M.hw(h), KEYS[k]) for h in hws for k in c["keys"].split(",")]
    return points


def _window(c, rng):
    return rng.randrange(_tilings(c) * 540000 - c["n"])


def prepare(case, seed):
    import torch
    rng = random.Random(seed)
    s = {"kind": case["kind"], "flags": M.SEARCH_EXHAUSTIVE if case.get("exhaustive") else M.SEARCH_PRUNED}
    if case["kind"] == "sweep":
        s["points"] = M.ManyPoints(_sweep(case, rng))
        return s
    s["attention"] = case["attention"]
    s["w"] = (M.workload if case["attention"] else M.chain)(_problem(case))
    s["h"] = M.hw(_hardware(case, rng))
    if case["kind"] in ("search", "noalloc"):
        s["keys"] = [KEYS[k] for k in case["keys"].split("+")]
    if case["kind"] == "noalloc":
        s["out"] = torch.zeros(38, dtype=torch.int32, device="cuda")
    if case["kind"] == "records":
        s["first"], s["n"] = _window(case, rng), case["n"]
        s["out"] = None if case["host"] else torch.empty((case["n"], 8), dtype=torch.int64, device="cuda")
        s["picks"] = [s["first"] + k * (case["n"] // 16) for k in range(16)]
    return s


def _records(results):
    """Mapping, cost and counts, and the two metrics once more, of result records, without their padding and times."""
    raw = np.frombuffer(results, dtype=np.int32).reshape(-1, 38)
    metrics = raw.view(np.float64)[:, 12:14]
    return {"mapping": raw[:, :13], "cost": raw[:, 14:34], "energy": metrics[:, 0], "latency": metrics[:, 1]}


def run(state):
    kind = state["kind"]
    if kind == "sweep":
        return _records(M.mmee_search_many(state["points"], state["flags"])[0])
    att, w, h = state["attention"], state["w"], state["h"]
    if kind == "search":
        call = M.mmee_search_multi if att else M.mmee_chain_search_multi
        return [_records(r) for r in call(w, h, state["keys"], state["flags"])]
    if kind == "pareto":
        return _records(b"".join((M.mmee_pareto if att else M.mmee_chain_pareto)(w, h, state["flags"])[1]))
    if kind == "front":
        return _records(b"".join((M.mmee_front_bs_da if att else M.mmee_chain_front_bs_da)(w, h, state["flags"])[1]))
    if kind == "noalloc":
        out = state["out"]
        M.mmee_search_noalloc(w, h, state["keys"][0], state["flags"], out.data_ptr())
        return {"mapping": out[:13], "cost": out[14:34]}
    records = M.mmee_eval_batch if att else M.mmee_chain_eval_batch
    if state["out"] is not None:
        records(w, h, state["first"], state["n"], state["out"].data_ptr())
        return state["out"]
    got = records(w, h, state["first"], state["n"])
    maps = (M.mmee_decode if att else M.mmee_chain_decode)(w, h, state["picks"])
    raw = got.view(np.int64).reshape(-1, 8)
    return {"records": raw, "energy": got["energy_pj"], "latency": got["latency_cycles"],
            "mappings": np.frombuffer(b"".join(maps), dtype=np.int32).reshape(-1, 14)[:, :13]}


def tolerance(case):
    # counts, mappings and index ties are whole numbers; energy and latency are formed in 64 bits in a fixed order
    return "exact"


def work(case):
    keys = len(case.get("keys", "energy").replace(",", "+").split("+"))
    if case["kind"] == "sweep":
        T = sum(_tilings(_attention(int(N), int(d), 1)) for N in case["Ns"].split(",") for d in case["ds"].split(",")) * case["n_hw"]
        n = case["n_hw"] * len(case["Ns"].split(",")) * len(case["ds"].split(",")) * keys
        return {"bytes": n * 400, "flops": T * (KEPT_ROWS * 5 + 18 * 2 * keys)}
    if case["kind"] == "records":
        return {"bytes": 64 * case["n"], "flops": 20 * case["n"]}
    T = _tilings(case)
    if case.get("exhaustive"):
        # per (row, tiling): two buffer sizes, their maximum, the capacity, traffic, its energy, the mask; per
        # stationary combination and key: one addition or maximum and the running minimum
        return {"bytes": 1024, "flops": T * DATAFLOW_ROWS * (8 + 9 * 2 * keys)}
    # per kept row the buffer sizes, traffic, mask and minimum; the 18 combinations once per tiling
    return {"bytes": 1024, "flops": T * (KEPT_ROWS * 5 + 18 * 2 * keys)}


# ---- the model in plain torch, 64 bits ------------------------------------------------------------
# Dimensions i=0, k=1, l=2, j=3; operands A(i,k) B(k,l) D(l,j) E(i,j), and C(i,l) between the two products.

OWN = {"A": (0, 1), "B": (1, 2), "D": (2, 3), "E": (0, 3)}


def _order(rank):
    left, out = [0, 1, 2, 3], []
    for f in (6, 2, 1, 1):
        out.append(left.pop(rank // f))
        rank %= f
    return out


def _loops(own, pos, nest, prefix, level):
    """Loops outside the operand that bring its block in again, as a bit mask."""
    outside = [x for x in own if pos[x] >= level]
    if not outside:
        return 0
    blocker = min(outside, key=lambda x: pos[x])
    counted = prefix if level == 0 and blocker in prefix else {x for x in nest if pos[x] >= pos[blocker]}
    return sum(1 << x for x in counted if x not in own)


def _row(levels, rank, r, f):
    """What a row fixes: per operand the loops its buffer spans and those that refetch it; None if it is no dataflow."""
    order = _order(rank)
    pos = {x: 3 - slot for slot, x in enumerate(order)}
    if r and (not f or pos[1] > pos[3]):
        return None
    prefix = set()
    for x in order:
        if x not in ({0, 2, 3} if r else {0, 2}):
            break
        prefix.add(x)
    nests = {"A": prefix | {0, 1, 2}, "B": prefix | {0, 1, 2}, "D": prefix | {0, 2, 3}, "E": prefix | {0, 2, 3}}
    spans, again, kept = [], [], []
    for name, level in zip("ABDE", levels):
        spans.append(sum(1 << x for x in OWN[name] if pos[x] < level))
        again.append(_loops(OWN[name], pos, nests[name], prefix, level))
        kept.append(int(level >= 1))
    c_span = sum(1 << x for x in (0, 2) if f and x not in prefix)
    spill = _loops((0, 2), pos, nests["A"], prefix, 0) & 2
    fetch = _loops((0, 2), pos, nests["D"], prefix, 0) & 8
    return (*spans, *again, *kept, c_span, -1 if f else spill, -1 if f else fetch)


class _Model:
    def __init__(self, case, hw):
        import torch
        self.t, self.c, self.h = torch, case, hw
        dev = "cuda" if torch.cuda.is_available() else "cpu"
        div = [_divisors(case[q], case["mode"]) for q in "IKLJ"]
        n = [len(v) for v in div]
        t = torch.arange(n[0] * n[1] * n[2] * n[3], device=dev)
        self.X = [case[q] for q in "IKLJ"]
        self.G, self.D = [], []
        for q in range(4):
            g = torch.tensor(div[q], dtype=torch.float64, device=dev)[t % n[q]]
            t = t // n[q]
            self.G.append(g)
            self.D.append(self.X[q] / g)
        one = torch.ones_like(self.G[0])
        prod = []
        for mask in range(16):
            v = one
            for q in range(4):
                v = v * self.D[q] if mask >> q & 1 else v
            prod.append(v)
        self.prod = torch.stack(prod)

    def rows(self, rows):
        """(buffer size, DRAM words) of rows x tilings."""
        G, X, idx = self.G, self.X, self.t.tensor(rows, device=self.prod.device)
        size = [self.prod[idx[:, k]] * (G[a] * G[b]) for k, (a, b) in enumerate(OWN.values())]
        c = self.prod[idx[:, 12]] * (G[0] * G[2])
        kept = [s * idx[:, 8 + k, None] for k, s in enumerate(size)]
        bs = self.t.maximum(size[0] + size[1] + c + kept[2] + kept[3], size[2] + size[3] + c + kept[0] + kept[1])
        da = sum(self.prod[idx[:, 4 + k]] * float(X[a] * X[b]) for k, (a, b) in enumerate(OWN.values()))
        unfused = (idx[:, 13] >= 0)[:, None]
        through = float(X[0] * X[2]) * (self.prod[idx[:, 13].clamp(min=0)] + self.prod[idx[:, 14].clamp(min=0)] + 2.0)
        return bs, da + self.t.where(unfused, through, self.t.zeros_like(through))

    def _tile(self, m, r, n, mode):
        h = self.h
        u, v, time = ((r, n, m), (m, r, n), (m, n, r))[mode]
        up = lambda a, b: self.t.ceil(a / b)  # noqa: E731
        words = u * v + time * u * up(v, h["pe_cols"] * (h["rf_bytes"] // 2 // 2)) + time * v * up(u, h["pe_rows"])
        return words, up(u, h["pe_rows"]) * up(v, h["pe_cols"]) * time

    def costs(self, da, r, s1, s2):
        """(energy, latency) of every row x tiling with recomputation r and stationary modes s1, s2."""
        h, G, D, X, BH = self.h, self.G, self.D, self.X, float(self.c["batch"])
        w1, c1 = self._tile(G[0], G[1], G[2], s1)
        w2, c2 = self._tile(G[0], G[2], G[3], s2)
        rho = D[3] if r else self.t.ones_like(D[3])
        n1, n2 = rho * D[0] * D[1] * D[2], D[0] * D[2] * D[3]
        br, comp = n1 * w1 + n2 * w2, n1 * c1 + n2 * c2
        mac, sm = rho * float(X[0] * X[1] * X[2]) + float(X[0] * X[2] * X[3]), rho * float(X[0] * X[2])
        e = h["e_dram"] * (BH * da) + h["e_gb"] * (BH * (da + br)) + h["e_rf"] * (BH * 3 * mac) + h["e_mac"] * (BH * (mac + self.c["c_softmax"] * sm))
        lat = self.t.maximum(self.t.maximum(comp.expand_as(da), da * 2.0 / h["dram_bw"]), br * 2.0 / h["gb_bw"]) * (BH / h["n_arrays"])
        return e, lat

    def every(self):
        """(energy, latency) of all feasible candidates, in pieces; rows with equal terms once."""
        for r, f in ((0, 0), (0, 1), (1, 1)):
            found = {_row((p % 5, p // 5 % 5, p // 25 % 5, p // 125), rank, r, f) for rank in range(24) for p in range(625)}
            rows = sorted(found - {None})
            step = max(1, (1 << 23) // self.prod.shape[1])
            for at in range(0, len(rows), step):
                bs, da = self.rows(rows[at:at + step])
                fits = bs * 2 <= self.h["gb_bytes"]
                for s in range(9):
                    e, lat = self.costs(da, r, s % 3, s // 3)
                    yield e[fits], lat[fits]


def exact(case, seed):
    rng = random.Random(seed)
    # fronts of whole numbers and records on the device hold no computed number of their own; of the
    # energy-delay optimum only the product is determined, not its factors
    if case["kind"] in ("sweep", "front", "noalloc") or "edp" in case.get("keys", ""):
        return None
    if (case["kind"] == "records" and not case["host"]) or (case["kind"] != "records" and _tilings(case) > 20000):
        return None
    m = _Model(case, _hardware(case, rng))
    t, T = m.t, _tilings(case)
    if case["kind"] == "records":
        first, n = _window(case, rng), case["n"]
        energy, latency = np.full(n, np.inf), np.full(n, np.inf)
        for row in range(first // T, (first + n - 1) // T + 1):
            p, rank, r, s1, s2, f = row % 625, row // 625 % 24, row // 15000 % 2, row // 30000 % 3, row // 90000 % 3, row // 270000
            terms = _row((p % 5, p // 5 % 5, p // 25 % 5, p // 125), rank, r, f)
            if terms is None:
                continue
            lo, hi = max(first, row * T), min(first + n, (row + 1) * T)
            bs, da = m.rows([terms])
            e, lat = m.costs(da, r, s1, s2)
            over = bs * 2 > m.h["gb_bytes"]
            for out, v in ((energy, e), (latency, lat)):
                out[lo - first:hi - first] = v.masked_fill(over, math.inf)[0, lo - row * T:hi - row * T].cpu().numpy()
        return {"records": None, "energy": energy, "latency": latency, "mappings": None}
    if case["kind"] == "pareto":
        front = t.empty((2, 0), dtype=t.float64, device=m.prod.device)
        for e, lat in m.every():
            low = t.cummin(front[1], 0).values if front.shape[1] else None
            if low is not None:             # drop what a front point already beats or equals
                at = t.searchsorted(front[0].contiguous(), lat, right=True) - 1
                new = (at < 0) | (e < low[at.clamp(min=0)])
                e, lat = e[new], lat[new]
            both = t.cat([front, t.stack([lat, e])], 1)
            both = both[:, t.sort(both[1], stable=True).indices]
            both = both[:, t.sort(both[0], stable=True).indices]
            low = t.cummin(both[1], 0).values if both.shape[1] else both[1]
            keep = t.ones(both.shape[1], dtype=t.bool, device=both.device)
            keep[1:] = both[1, 1:] < low[:-1]
            front = both[:, keep]
        return {"mapping": None, "cost": None, "energy": front[1].cpu().numpy(), "latency": front[0].cpu().numpy()}
    best = {}
    for e, lat in m.every():
        if not e.numel():
            continue
        for key in case["keys"].split("+"):
            v = e if key == "energy" else lat
            low = v.min()
            second = (lat if key == "energy" else e)[v == low].min()
            best[key] = min(best.get(key, (math.inf, math.inf)), (low.item(), second.item()))
    # ties of one metric are broken by index, so the other metric has a value of its own only under the lexicographic key
    out = []
    for key in case["keys"].split("+"):
        first, second = np.array([best[key][0]]), np.array([best[key][1]])
        out.append({"energy": {"energy": first, "latency": None}, "latency": {"energy": None, "latency": first},
                    "latency_then_energy": {"energy": second, "latency": first}}[key] | {"mapping": None, "cost": None})
    return out
