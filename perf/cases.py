"""Performance cases of the streaming KV step and of the adaptation objective.

Two families, each through the library's public calls:

* streaming steps (``kind`` "unit"): a cache filled by earlier one-second units
  (append + eviction under a budget, transcript rows kept), then per pass ONE
  step: the new rows of every stream are appended, attended and the budget
  check evicts, over all layers of the cache.  ``calls`` picks the entry points:
  "fused" (a2t_append_attn per layer), "split" (a2t_append + a2t_chunk_attn per
  layer, a2t_decode_attn for single rows), "graph" (device-planned steps, one
  HIP graph replay per step).  A pass returns the attention output, the evicted
  counts and the K and V pools.
* the adaptation objective (``kind`` "distill"): one evaluation of the masked
  cross-entropy, the temperature-scaled divergence and the group-balanced means,
  with or without the gradient.

The steps of the timed passes carry evictable rows (audio, markers, delimiters);
with ``text`` > 0 every fourth unit also carries transcript rows.  Transcript rows
are never evicted, so without them a session stays at its budget for any number
of passes.
"""
import ctypes as C
import functools
import math
import zlib

import numpy as np
import torch

import paper_2609_31224_amd as a2t

DEV = "cuda:0"
SLOTS = 4            # prepared units a session cycles through
THETA = 1.0e6
ACOUSTIC, DELIM, TEXT = a2t.SEG_ACOUSTIC, a2t.SEG_DELIM, a2t.SEG_TEXT
# a listening unit with t transcript rows
UNITS = [np.array([ACOUSTIC] * 17 + [DELIM] + [TEXT] * t + [DELIM], np.uint8) for t in range(65)]


def listed():
    def unit(name, **kw):
        c = dict(name=name, kind="unit", dtype="bf16", layers=4, streams=1, hq=32, hkv=8, d=128,
                 budget=4096, even=True, window=30, rows=22, text=0, calls="fused")
        c.update(kw)
        return c

    return [
        # the smallest session: one layer, four query heads over one KV head, fp32
        unit("tiny_f32_unit", dtype="f32", layers=1, hq=4, hkv=1, d=64, budget=256, window=3),
        # a ten-minute session's unit step over a whole 36-layer model
        unit("stream_unit", layers=36, text=3),
        # batched listening: sessions of unequal length, residency from an eighth of 4096 up
        unit("varlen_units", streams=21, even=False),
        # speaking: 64 sessions decode one row each
        unit("decode_batch", streams=64, rows=1),
        # one side-channel token of one session: a single row, append and decode as two calls
        unit("side_channel_row", rows=1, calls="split"),
        # hour-long sessions under a larger budget
        unit("hour_units", streams=16, budget=8192, window=60),
        # a long chunk fed at once onto a resident session (the most rows one step takes)
        unit("catch_up_chunk", rows=1024, window=0),
        # a prompt chunk of odd length onto an empty cache, head dim 64
        unit("prompt_chunk", rows=777, d=64, hkv=4, budget=0, window=0, calls="split"),
        # the fp32 storage type at the model's heads
        unit("f32_units", dtype="f32", streams=2, budget=2048),
        # device-planned steps, captured once and replayed per unit
        unit("graph_units", layers=8, streams=2, calls="graph"),
        # side-channel training batch: 16 utterances of 12 units, the whole vocabulary, gradient
        dict(name="distill_grad", kind="distill", dtype="bf16", utterances=16, units=12, vocab=151936,
             added=2, temperature=1.0, grad=True),
        # validation loss of a small batch: fp32 logits, odd vocabulary, softened distributions
        dict(name="distill_loss_f32", kind="distill", dtype="f32", utterances=4, units=9, vocab=32003,
             added=2, temperature=2.0, grad=False),
    ]


def draw(rng):
    """One more case of the same ranges; sizes log-uniform, odd ones among them."""
    def log_int(lo, hi):
        return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))

    if rng.random() < 0.3:
        dtype = rng.choice(["bf16", "f32"])
        return dict(kind="distill", dtype=dtype, utterances=log_int(1, 12), units=log_int(2, 12),
                    vocab=log_int(1000, 152000 if dtype == "bf16" else 80000), added=rng.choice([1, 2, 7]),
                    temperature=rng.choice([0.5, 1.0, 2.0]), grad=rng.random() < 0.7)
    hkv = rng.choice([1, 2, 4, 8])
    c = dict(kind="unit", dtype="bf16", layers=rng.choice([1, 2, 4]), streams=1,
             hq=min(32, hkv * rng.choice([1, 2, 4, 8])),
             hkv=hkv, d=rng.choice([64, 128]), budget=log_int(200, 8192), even=True, window=rng.choice([1, 3, 30]),
             rows=rng.choice([1, 17, 22, log_int(2, 90)]), text=0, calls=rng.choice(["fused", "fused", "split", "graph"]))
    shape = rng.random()
    if shape < 0.25:      # a long chunk, onto a session or onto an empty cache
        c.update(rows=log_int(91, 1024), window=0, budget=rng.choice([0, log_int(200, 4096)]),
                 calls=rng.choice(["fused", "split"]))
    elif shape < 0.7:     # a batch of sessions
        most = 64 if c["rows"] == 1 else max(3, min(21, 460 // c["rows"]))
        c.update(streams=log_int(2, most), even=rng.random() < 0.4,
                 budget=min(c["budget"], 4096))
    if c["calls"] != "graph" and rng.random() < 0.3:
        c.update(dtype="f32", streams=min(c["streams"], 4), budget=min(c["budget"], 2048), rows=min(c["rows"], 128))
    if c["calls"] == "graph":
        c.update(streams=min(c["streams"], 16))
    return c


# ------------------------------------------------------------------ the session's structure
def _layout(case):
    return _layout_of(tuple(sorted((k, v) for k, v in case.items() if k != "name")))


@functools.lru_cache(maxsize=32)
def _layout_of(key):
    """What a case's sessions hold, from the case alone: per stream the budget, the fill
    (one array of row classes per unit), the rows that survive it, and the timed units."""
    case = dict(key)
    rng = np.random.default_rng(zlib.crc32(repr(key).encode()))
    S, B, window = case["streams"], case["budget"], case["window"]
    budgets = [B] * S if case["even"] else [int(x) for x in rng.integers(B // 8, B + 1, size=S)]
    fill, alive = [], []
    for s in range(S):
        # one quarter more units than the budget holds, so that some have been evicted; a
        # session that is emptied after every step starts empty
        n_units = 0 if budgets[s] == 0 else int(1.25 * budgets[s] / 22) + window + 1
        texts = [int(t) for t in np.minimum(rng.poisson(3.0, size=n_units), 64)]
        fill.append([UNITS[t] for t in texts])
        resident, oldest = 0, 0
        for u, t in enumerate(texts):
            resident += 19 + t
            while resident > budgets[s] and oldest <= u - window:
                resident -= 19
                oldest += 1
        unit = np.repeat(np.arange(n_units), [19 + t for t in texts])
        seg = np.concatenate(fill[s]) if n_units else np.zeros(0, np.uint8)
        alive.append(np.flatnonzero((unit >= oldest) | (seg == TEXT)))
    steps = max(len(u) for u in fill)
    # streams start at different steps so that all fills end together
    first = [steps - len(u) for u in fill]
    timed = []
    for j in range(SLOTS):
        segs = []
        for s in range(S):
            n = case["rows"]
            if 4 < n < 91:   # ordinary units differ in length; single rows and long chunks do not
                n += int(rng.integers(-3, 4))
            t = int(rng.poisson(case["text"])) if case["text"] and j == 0 else 0
            segs.append(np.array([ACOUSTIC] * n + [TEXT] * t, np.uint8))
        timed.append(segs)
    return budgets, fill, first, steps, alive, timed


def _values(case, seed):
    """The seeded generator of every K, V and Q value, in the order both users draw them."""
    g = torch.Generator(device=DEV)
    g.manual_seed(seed)
    dt = torch.float32 if case["dtype"] == "f32" else torch.bfloat16

    def rand(rows, heads):
        return torch.randn((case["layers"], rows, heads, case["d"]), generator=g, device=DEV).to(dt)
    return rand


def _fill_steps(case, lay):
    """(streams of the step, their row classes) for every fill step."""
    _, fill, first, steps, _, _ = lay
    for t in range(steps):
        ids = [s for s in range(case["streams"]) if t >= first[s]]
        yield t, ids, [fill[s][t - first[s]] for s in ids]


def _i32(x):
    return (C.c_int32 * len(x))(*[int(v) for v in x])


class Session:
    """A filled cache and the units that the passes feed it."""

    def __init__(self, case, seed):
        self.case = case
        lay = _layout(case)
        budgets, fill, first, _, _, timed = lay
        S, L, D, hq, hkv = case["streams"], case["layers"], case["d"], case["hq"], case["hkv"]
        self.S, self.L = S, L
        rows_fill = [sum(len(u) for u in f) for f in fill]
        kept = max(sum(int((u == TEXT).sum()) for u in f) for f in fill) + 64
        if case["text"]:
            kept += 16384
        longest = max([len(x) for segs in timed for x in segs] + [len(u) for f in fill for u in f])
        self.graph = case["calls"] == "graph"
        unit_rows = max(budgets) + longest * (case["window"] + 2) + 64
        dt = torch.float32 if case["dtype"] == "f32" else torch.bfloat16
        shape = (L * S * hkv * (unit_rows + kept) * D,)
        self.k_pool = torch.zeros(shape, dtype=dt, device=DEV)
        self.v_pool = torch.zeros(shape, dtype=dt, device=DEV)
        self.stream = torch.cuda.current_stream()
        self.cache = a2t.a2t_cache_create(
            L, S, hq, hkv, D, a2t.A2T_F32 if case["dtype"] == "f32" else a2t.A2T_BF16, unit_rows, kept,
            longest, rope_theta=THETA, stream=self.stream, k_pool=self.k_pool, v_pool=self.v_pool)
        self.lib, self.h = a2t.raw_lib(), self.cache.ptr
        rand = _values(case, seed)
        pos = np.zeros(S, np.int64)
        for t, ids, segs in _fill_steps(case, lay):
            n = [len(x) for x in segs]
            k, v = rand(sum(n), hkv), rand(sum(n), hkv)
            at = np.concatenate([np.arange(pos[s], pos[s] + m) for s, m in zip(ids, n)])
            unit = [t - first[s] for s in ids]
            a2t.a2t_append(self.cache, a2t.A2T_ALL_LAYERS, ids, n, k, v, np.concatenate(segs), at, unit)
            a2t.a2t_evict(self.cache, ids, [budgets[s] for s in ids], case["window"])
            pos[ids] += n
        self.next_unit = np.array([len(f) for f in fill], np.int32)
        self.next_pos = pos.astype(np.int32)
        self.window = case["window"]
        self.ids, self.budget = _i32(range(S)), _i32(budgets)
        self.evicted, self.unmet = np.zeros(S, np.int32), np.zeros(S, np.uint8)
        self.slots = []
        stride = longest if self.graph else 0
        for segs in timed:
            n = [len(x) for x in segs]
            q, k, v = rand(sum(n), hq), rand(sum(n), hkv), rand(sum(n), hkv)
            if self.graph:   # listed stream i's rows start at row i * max_step_rows
                place = torch.from_numpy(np.concatenate([i * stride + np.arange(m) for i, m in enumerate(n)])).to(DEV)

                def spread(x):
                    y = torch.zeros((L, S * stride) + x.shape[2:], dtype=x.dtype, device=DEV)
                    y[:, place] = x
                    return y
                q, k, v = spread(q), spread(k), spread(v)
            self.slots.append(Slot(self, segs, q, k, v, torch.zeros_like(q), stride))
        self.count = 0
        if self.graph:
            self._capture(budgets, stride)
        torch.cuda.synchronize()

    def _capture(self, budgets, stride):
        """Device-planned steps: one graph per prepared unit, with the step's positions and
        unit ids advanced by the graph itself."""
        S = self.S
        self.d_next = torch.from_numpy(self.next_pos).to(DEV)
        self.d_unit = torch.from_numpy(self.next_unit).to(DEV)
        self.d_pos = torch.zeros((S, stride), dtype=torch.int32, device=DEV)
        self.d_budget = torch.tensor(budgets, dtype=torch.int32, device=DEV)
        self.d_evicted = torch.zeros(S, dtype=torch.int32, device=DEV)
        a2t.a2t_dev_begin(self.cache)
        side = torch.cuda.Stream()
        side.wait_stream(self.stream)
        torch.cuda.synchronize()
        a2t.a2t_set_stream(self.cache, side)
        for s in self.slots:
            s.graph = torch.cuda.CUDAGraph()
            with torch.cuda.graph(s.graph, stream=side):
                torch.add(self.d_next.unsqueeze(1), s.d_rel, out=self.d_pos)
                a2t.a2t_dev_open(self.cache, list(range(S)), s.d_n, self.d_unit, s.d_seg, self.d_pos)
                for layer in range(self.L):
                    a2t.a2t_dev_append_attn(self.cache, layer, s.k[layer], s.v[layer], s.q[layer], s.o[layer])
                a2t.a2t_dev_evict(self.cache, self.d_budget, self.window, self.d_evicted)
                self.d_next.add_(s.d_n)
                self.d_unit.add_(1)
        a2t.a2t_set_stream(self.cache, self.stream)
        torch.cuda.synchronize()

    def step(self):
        s = self.slots[self.count % SLOTS]
        self.count += 1
        if self.graph:
            s.graph.replay()
            return {"o": s.o, "evicted": self.d_evicted, "k": self.k_pool, "v": self.v_pool}
        lib, h, S = self.lib, self.h, self.S
        np.add(s.rel, self.next_pos[s.of], out=s.pos)
        unit = a2t_ptr(self.next_unit)
        single, calls = s.single, self.case["calls"]
        for layer in range(self.L):
            seg, pos, uid = (s.p_seg, s.p_pos, unit) if layer == 0 else (None, None, None)
            if calls == "fused":
                rc = lib.a2t_append_attn(h, layer, S, self.ids, s.n, s.p_k[layer], s.p_v[layer], seg, pos, uid,
                                         s.n, s.p_q[layer], s.p_o[layer])
            else:
                rc = lib.a2t_append(h, layer, S, self.ids, s.n, s.p_k[layer], s.p_v[layer], seg, pos, uid)
                if not rc:
                    rc = (lib.a2t_decode_attn(h, layer, S, self.ids, s.p_q[layer], s.p_o[layer]) if single else
                          lib.a2t_chunk_attn(h, layer, S, self.ids, s.n, s.p_q[layer], s.p_o[layer]))
            if rc:
                raise a2t.A2TError(rc, "step")
        rc = lib.a2t_evict(h, S, self.ids, self.budget, self.window, a2t_ptr(self.evicted),
                           self.unmet.ctypes.data_as(C.POINTER(C.c_uint8)))
        if rc:
            raise a2t.A2TError(rc, "a2t_evict")
        self.next_unit += 1
        self.next_pos += s.counts
        return {"o": s.o, "evicted": self.evicted.copy(), "k": self.k_pool, "v": self.v_pool}

    def __del__(self):
        cache = getattr(self, "cache", None)
        if cache is not None:
            torch.cuda.synchronize()
            a2t.a2t_cache_destroy(cache)


def a2t_ptr(x):
    return x.ctypes.data_as(C.POINTER(C.c_int32))


class Slot:
    """One prepared unit: its rows of every stream and the marshalled arguments."""

    def __init__(self, session, segs, q, k, v, o, stride):
        n = [len(x) for x in segs]
        self.q, self.k, self.v, self.o = q, k, v, o
        self.single = all(m == 1 for m in n)
        self.counts = np.array(n, np.int32)
        if stride:
            self.d_n = torch.from_numpy(self.counts).to(DEV)
            self.d_rel = torch.arange(stride, dtype=torch.int32, device=DEV).unsqueeze(0).repeat(len(n), 1)
            seg = np.zeros((len(n), stride), np.uint8)
            for i, x in enumerate(segs):
                seg[i, :len(x)] = x
            self.d_seg = torch.from_numpy(seg).to(DEV)
            return
        self.n = _i32(n)
        self.of = np.repeat(np.arange(len(n)), n)
        self.rel = np.concatenate([np.arange(m, dtype=np.int32) for m in n])
        self.pos = np.zeros_like(self.rel)
        self.seg = np.concatenate(segs)
        self.p_pos, self.p_seg = a2t_ptr(self.pos), self.seg.ctypes.data_as(C.POINTER(C.c_uint8))
        self.p_q, self.p_k, self.p_v, self.p_o = ([x[i].data_ptr() for i in range(session.L)] for x in (q, k, v, o))


# ------------------------------------------------------------------ the objective's batch
def _rows(case):
    """Kinds, targets and groups of a batch's rows (the side channel's call order per unit)."""
    rng = np.random.default_rng([case["utterances"], case["units"], case["vocab"]])
    V, A = case["vocab"], case["added"]
    out = []
    for _ in range(case["utterances"] * case["units"]):
        out.append((a2t.A2T_ROW_NATIVE, -1, int(rng.choice(3, p=[0.8, 0.1, 0.1])), -1))
        text = [int(x) for x in rng.integers(0, V, size=min(rng.poisson(3.0), 64))]
        out += [(a2t.A2T_ROW_ASR, y, -1, -1) for y in [V] + text + [V + A - 1]]
        out += [(a2t.A2T_ROW_NATIVE, -1, -1, int(rng.random() < 0.2)) for _ in range(rng.poisson(1.0))]
    kind, target, dec, turn = zip(*out)
    return np.array(kind, np.int8), np.array(target, np.int32), np.array(dec, np.int8), np.array(turn, np.int8)


def _logits(case, seed, n):
    g = torch.Generator(device=DEV)
    g.manual_seed(seed)
    V, A = case["vocab"], case["added"]
    dt = torch.float32 if case["dtype"] == "f32" else torch.bfloat16
    teacher = torch.zeros((n, -(-V // 8) * 8), device=DEV, dtype=dt)
    student = torch.zeros((n, -(-(V + A) // 8) * 8), device=DEV, dtype=dt)
    t = torch.randn((n, V), generator=g, device=DEV).mul_(2.0)
    teacher[:, :V] = t
    student[:, :V] = t.add_(torch.randn((n, V), generator=g, device=DEV), alpha=0.5)
    student[:, V:V + A] = torch.randn((n, A), generator=g, device=DEV).sub_(2.0)
    return student, teacher


class Batch:
    """One batch of the objective: its logits, row metadata and handle."""

    def __init__(self, case, seed):
        self.case, self.meta = case, _rows(case)
        n = len(self.meta[0])
        self.student, self.teacher = _logits(case, seed, n)
        self.losses = torch.zeros(5, device=DEV)
        self.grad = torch.zeros_like(self.student) if case["grad"] else None
        self.handle = a2t.a2t_distill_create(
            n, case["vocab"], case["added"], a2t.A2T_F32 if case["dtype"] == "f32" else a2t.A2T_BF16,
            stream=torch.cuda.current_stream())

    def step(self):
        a2t.a2t_distill_loss(self.handle, self.student, self.teacher, *self.meta, self.case["temperature"],
                             self.losses, self.grad)
        out = {"losses": self.losses}
        if self.grad is not None:
            out["grad"] = self.grad[:, :self.case["vocab"] + self.case["added"]]
        return out

    def __del__(self):
        handle = getattr(self, "handle", None)
        if handle is not None:
            a2t.a2t_distill_destroy(handle)


# ------------------------------------------------------------------ the interface
def prepare(case, seed):
    return Session(case, seed) if case["kind"] == "unit" else Batch(case, seed)


def run(state):
    return state.step()


def work(case):
    """Least bytes and operations of a pass.  A step reads every resident K and V row of
    its streams once, and reads Q and the new K and V and writes O and the rows once; its
    products cover the visible keys.  The objective reads the student's logits of every
    row and the teacher's of the native rows, and writes the gradient."""
    if case["kind"] == "distill":
        kind = _rows(case)[0]
        e = 4 if case["dtype"] == "f32" else 2
        vs = case["vocab"] + case["added"]
        n, native = len(kind), int((kind == a2t.A2T_ROW_NATIVE).sum())
        return {"bytes": e * (n * vs + native * case["vocab"] + (n * vs if case["grad"] else 0)),
                "flops": 8.0 * n * vs}
    lay = _layout(case)
    e = 4 if case["dtype"] == "f32" else 2
    D, hq, hkv = case["d"], case["hq"], case["hkv"]
    by = fl = 0.0
    for segs in lay[5]:
        for alive, seg in zip(lay[4], segs):
            m, R = len(seg), len(alive) + len(seg)
            by += e * D * (2 * hkv * R + 2 * hkv * m + 2 * hq * m)
            fl += 4.0 * D * hq * (m * (R - m) + m * (m + 1) / 2)
    return {"bytes": case["layers"] * by / SLOTS, "flops": case["layers"] * fl / SLOTS}


def tolerance(case):
    """Four times what the path differs from 64 bits by: fp32 outputs 2e-7 to 3e-7 (sums of up
    to 10^4 terms), bf16 outputs 3.5e-3 (outputs, probabilities and rotated keys are rounded
    to 8 bits of mantissa)."""
    if case["dtype"] == "f32":
        return {"rel": 1.2e-6, "max": 5e-5}
    return {"rel": 1.2e-2, "max": 0.1}


def exact(case, seed):
    return _exact_distill(case, seed) if case["kind"] == "distill" else _exact_unit(case, seed)


def _rotate(x, pos):
    """Rotate-half rotary encoding of x [..., rows, heads, D] at the rows' positions, in 64 bits."""
    half = x.shape[-1] // 2
    inv = THETA ** (-2.0 * torch.arange(half, dtype=torch.float64, device=DEV) / x.shape[-1])
    ang = pos.to(torch.float64)[:, None] * inv
    c, s = torch.cos(ang)[:, None, :], torch.sin(ang)[:, None, :]
    lo, hi = x[..., :half], x[..., half:]
    return torch.cat([lo * c - hi * s, hi * c + lo * s], -1)


def _exact_unit(case, seed):
    """The first pass: attention of its rows over the rows that the fill left and themselves."""
    lay = _layout(case)
    budgets, fill, first, _, alive, timed = lay
    S, L, D, hq, hkv = case["streams"], case["layers"], case["d"], case["hq"], case["hkv"]
    rand = _values(case, seed)
    ks, vs = [[] for _ in range(S)], [[] for _ in range(S)]
    for _, ids, segs in _fill_steps(case, lay):
        n = [len(x) for x in segs]
        k, v = rand(sum(n), hkv), rand(sum(n), hkv)
        for s, a, b in zip(ids, k.split(n, 1), v.split(n, 1)):
            ks[s].append(a)
            vs[s].append(b)
    outs, evicted = [], []
    n = [len(x) for x in timed[0]]
    q, k, v = rand(sum(n), hq), rand(sum(n), hkv), rand(sum(n), hkv)
    for s, (qs, kn, vn) in enumerate(zip(q.split(n, 1), k.split(n, 1), v.split(n, 1))):
        m = n[s]
        total = sum(len(u) for u in fill[s])
        keep = torch.from_numpy(np.concatenate([alive[s], total + np.arange(m)])).to(DEV)
        kk, vv = torch.cat(ks[s] + [kn], 1)[:, keep], torch.cat(vs[s] + [vn], 1)[:, keep]
        R = len(keep)
        mask = torch.arange(R, device=DEV)[None, :] > (R - m + torch.arange(m, device=DEV))[:, None]
        o = torch.empty((L, m, hq, D), dtype=torch.float64, device=DEV)
        for layer in range(L):
            kr = _rotate(kk[layer].double(), keep).permute(1, 2, 0).contiguous()       # [hkv, D, R]
            vr = vv[layer].double().permute(1, 0, 2).contiguous()                      # [hkv, R, D]
            qr = _rotate(qs[layer].double(), keep[-m:]).permute(1, 0, 2)               # [hq, m, D]
            for g in range(hkv):
                G = hq // hkv
                sc = torch.matmul(qr[g * G:(g + 1) * G].reshape(G * m, D), kr[g]).view(G, m, R) / math.sqrt(D)
                p = torch.softmax(sc.masked_fill_(mask, -math.inf), -1)
                o[layer, :, g * G:(g + 1) * G] = torch.matmul(p.view(G * m, R), vr[g]).view(G, m, D).permute(1, 0, 2)
        outs.append(o)
    o = torch.cat(outs, 1)
    if case["calls"] == "graph":
        stride = max([len(x) for segs in timed for x in segs] + [len(u) for f in fill for u in f])
        full = torch.zeros((L, S * stride, hq, D), dtype=torch.float64, device=DEV)
        at = np.concatenate([i * stride + np.arange(m) for i, m in enumerate(n)])
        full[:, torch.from_numpy(at).to(DEV)] = o
        o = full
    return {"o": o, "evicted": None, "k": None, "v": None}


def _exact_distill(case, seed):
    kind, target, dec, turn = (torch.from_numpy(x).to(DEV) for x in _rows(case))
    n, V, T = len(kind), case["vocab"], case["temperature"]
    vs = V + case["added"]
    student, teacher = _logits(case, seed, n)
    asr, nat = kind == a2t.A2T_ROW_ASR, kind == a2t.A2T_ROW_NATIVE
    w_asr, w_nat = asr.double() / asr.sum().clamp(min=1), nat.double() / nat.sum().clamp(min=1)

    def balanced(groups, count):
        members = [nat & (groups == g) for g in range(count)]
        members = [m for m in members if bool(m.any())]
        return sum((m.double() / (len(members) * m.sum()) for m in members), torch.zeros_like(w_nat))
    w_dec, w_turn = balanced(dec, 3), balanced(turn, 2)
    wk = w_nat + w_dec + w_turn
    ce, kl = torch.zeros(n, dtype=torch.float64, device=DEV), torch.zeros(n, dtype=torch.float64, device=DEV)
    grad = torch.zeros((n, vs), dtype=torch.float64, device=DEV) if case["grad"] else None
    for i in range(0, n, 64):
        r = slice(i, i + 64)
        s, t = student[r, :vs].double(), teacher[r, :V].double()
        l1, lt, lw = (torch.log_softmax(x, -1) for x in (s, s / T, t / T))
        hot = target[r].long().clamp(min=0)[:, None]
        ce[r] = torch.where(asr[r], -l1.gather(1, hot)[:, 0], 0.0)
        kl[r] = torch.where(nat[r], T * T * (lw.exp() * (lw - lt[:, :V])).sum(-1), 0.0)
        if grad is not None:
            d = lt.exp()
            d[:, :V] -= lw.exp()
            one = torch.zeros_like(s).scatter_(1, hot, 1.0)
            grad[r] = (wk[r] * T)[:, None] * d + w_asr[r][:, None] * (l1.exp() - one)
    parts = torch.stack([(w_asr * ce).sum(), (w_nat * kl).sum(), (w_dec * kl).sum(), (w_turn * kl).sum()])
    out = {"losses": torch.cat([parts, parts.sum()[None]])}
    if grad is not None:
        out["grad"] = grad
    return out
