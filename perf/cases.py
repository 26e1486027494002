"""The calls that are timed: the trace pipeline and its derived calls over the
range of traces this package serves.

A case names an entry point ("call") and the run whose trace it works on:
GPUs x iterations x layers of a Llama-shaped FSDP training run (per layer 14
forward and 14 backward kernels, `k_opt` optimizer kernels, one all-gather and
one reduce-scatter beside them), the number of compute streams, the marker
depth (4: iteration / phase / layer / operation; 6: sub-operation markers as
well, varying from iteration to iteration, one marker in a hundred lost), the
counter columns per record, and the order in which the records arrive:

    profiler   grouped by GPU, in start order (one file per rank, appended)
    merged     all ranks merged by time
    shuffled   records and markers in no order

Calls:

    step          Pipeline.step: alignment, attribution, overlap, aggregation
                  at every level, ratios, window fractions
    filter        the aggregation of a selection of iterations (and GPUs) of
                  a trace that is already aligned, with its ratios
    views         per-phase / per-operation tables, medians, throughput
    op_stats      overlap statistics and overhead breakdown per operation
    join          counters of seven serialized profiling passes attached to
                  the records
    launch_split  launch overhead split into preparation and call
"""
import math

import numpy as np
import torch

import paper_2512_08242_amd as ch

T0 = 1_700_000_000_000_000_000          # epoch-scale timestamps, ns
PHASES, OPS, WARMUP = 3, 64, 10
PASSES = (3, 3, 2, 2, 2, 2, 2)          # counter columns of each pass

# forward operations of a layer: class and number of kernels
# (0 GEMM, 1 attention, 2 elementwise, 3 RMSNorm, 4 RoPE, 5 all-gather,
# 6 reduce-scatter, 7 optimizer)
_FWD = [(3, 1), (0, 2), (4, 1), (1, 1), (0, 1), (2, 1), (3, 1), (0, 1),
        (2, 1), (0, 1), (2, 1), (0, 1), (2, 1)]
_MEAN_NS = [400e3, 300e3, 20e3, 30e3, 20e3, 0.0, 0.0, 5e3]
# events per microsecond of counters 1..12, by class
_RATE = [
    [1500, 300, 50, 2.0e6, 6.0e5, 4e3, 1e3, 20, 600, 300, 1.0e9, 40],
    [900, 900, 80, 1.5e6, 4.0e5, 3e3, 8e2, 60, 900, 400, 6.0e8, 30],
    [0, 1500, 60, 3.5e6, 3.5e6, 1e3, 3e3, 0, 10, 900, 0.0, 60],
    [0, 1400, 70, 3.0e6, 2.5e6, 1e3, 2e3, 5, 200, 800, 0.0, 50],
    [0, 1300, 60, 3.0e6, 3.0e6, 1e3, 2e3, 0, 50, 800, 0.0, 50],
    [0, 200, 40, 4.0e6, 4.0e6, 5e2, 4e3, 0, 0, 700, 0.0, 20],
    [0, 600, 40, 4.0e6, 4.0e6, 5e2, 4e3, 0, 0, 700, 0.0, 20],
    [0, 1200, 90, 2.5e6, 2.5e6, 1e3, 2e3, 0, 0, 600, 0.0, 30]]


def _case(name, call, gpus, iters, layers, k_opt=66, streams=1, depth=4,
          counters=16, order="profiler", **more):
    return dict(name=name, call=call, gpus=gpus, iters=iters, layers=layers,
                k_opt=k_opt, streams=streams, depth=depth, counters=counters,
                order=order, **more)


def listed():
    return [
        # two iterations of a small model on one GPU: what a developer looks
        # at while instrumenting; launches and host waits count (2,000 records)
        _case("step 1x2x4", "step", 1, 2, 4, k_opt=220, counters=0),
        # ten iterations of one node without hardware counters (245,760)
        _case("step 8x10x32", "step", 8, 10, 32, counters=0),
        # an ordinary profiled run: a hundred iterations, 16 counters (2.46M)
        _case("step 8x100x32", "step", 8, 100, 32),
        # a long run, the benchmark's trace (19.66M records, 7.2M rows)
        _case("step 8x800x32", "step", 8, 800, 32),
        # two compute and two communication streams per GPU, deep markers,
        # some of them lost (2.46M)
        _case("step 8x100x32 streams", "step", 8, 100, 32, streams=2,
              depth=6),
        # ranks merged by time, odd sizes, few counters (681,175 records)
        _case("step 5x61x29 merged", "step", 5, 61, 29, k_opt=47,
              counters=7, order="merged"),
        # the largest and least ordered trace: records and markers in no
        # order, four streams, deep markers (50.0M records, 37.9M markers)
        _case("step 8x2035x32 shuffled", "step", 8, 2035, 32, streams=2,
              depth=6, order="shuffled"),
        # statistics leave the warm-up iterations out: the aggregation of the
        # iterations past the tenth of an ordinary run (2.46M records)
        _case("filter 8x100x32", "filter", 8, 100, 32, level=255, lo=WARMUP,
              hi=99, few=False),
        # the figures' tables and medians of the long run
        _case("views 8x800x32", "views", 8, 800, 32),
        _case("op_stats 8x800x32", "op_stats", 8, 800, 32),
        # sixteen counters from seven profiling passes (9.83M records)
        _case("join 8x400x32", "join", 8, 400, 32),
        # preparation / call split of the long run's launch overhead
        _case("launch_split 8x800x32", "launch_split", 8, 800, 32,
              counters=0),
    ]


def draw(rng):
    def spread(lo, hi):
        return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))

    call = rng.choice(["step", "step", "step", "step", "filter", "views",
                       "op_stats", "join", "launch_split"])
    order = rng.choice(["profiler", "profiler", "profiler", "merged",
                        "shuffled"])
    gpus, layers, k_opt = rng.randint(1, 8), spread(2, 80), spread(5, 130)
    streams = rng.choice([1, 1, 2])
    depth = rng.choice([4, 4, 6])
    counters = rng.choice([0, 16, 16, rng.randint(1, 15)])
    most = 20_000_000 if order == "profiler" else 10_000_000
    records = spread(1000, most)
    iters = max(1, min(3000, records // (gpus * layers * (30 + k_opt))))
    layers = max(1, min(layers, most // (gpus * iters * (30 + k_opt))))
    c = _case("", call, gpus, iters, layers, k_opt, streams, depth, counters,
              order)
    del c["name"]
    if call == "join":
        c["counters"] = 16
    if call == "filter":
        c["lo"] = rng.randint(0, max(0, iters // 2))
        c["hi"] = rng.randint(c["lo"], iters)
        c["few"] = rng.random() < 0.3
        c["level"] = rng.choice([255, 255, 3, 2, 100])
    return c


# --------------------------------------------------------------------------
# Traces, made on the GPU
# --------------------------------------------------------------------------
class Trace(ch.DeviceTrace):
    """A trace of `case`, made in device memory from `seed`.

    The run's schedule -- when kernels start and ranges open -- belongs to
    the case, on a reference clock that ticks every 10 ns (a 100 MHz
    timestamp counter), so that the numbers of markers and rows are the
    case's.  The seed makes everything measured: how long each kernel takes
    within its slot, each GPU's clock and the moment it begins, the anchors,
    the counters, and the order of shuffled input."""

    def __init__(self, case, seed):
        dev = torch.device("cuda")
        g = torch.Generator(device=dev)
        g.manual_seed(seed)
        plan = torch.Generator(device=dev)
        plan.manual_seed(2512)
        G, I, L = case["gpus"], case["iters"], case["layers"]
        S, deep = case["streams"], case["depth"] > 4
        i64, u8 = torch.int64, torch.uint8
        rand = lambda *s, of=g: torch.rand(*s, generator=of, device=dev,
                                           dtype=torch.float64)
        tick = lambda v: v.mul(0.1).round_().to(i64).mul_(10)
        wait = lambda *s: tick(rand(*s, of=plan).clamp_(min=1e-12).log_()
                               .mul_(-5e3))      # launch gaps: 5 us mean
        self.n_gpus, self.depth = G, case["depth"]

        # ---- compute kernels: a timeline per (GPU, iteration, phase, layer)
        fwd = [(c, k, j) for j, (c, k) in enumerate(_FWD)]
        bwd = [(c, k, 16 + j) for j, (c, k) in reversed(list(enumerate(_FWD)))]
        opt = [(7, 3, 32), (7, case["k_opt"] - 3, 33)]
        ph = []
        for p, ops in enumerate((fwd, bwd, opt)):
            cls = [c for c, k, _ in ops for _ in range(k)]
            lab = [v for _, k, v in ops for _ in range(k)]
            op = [o for o, (_, k, _) in enumerate(ops) for _ in range(k)]
            K = len(cls)
            mean = torch.tensor([_MEAN_NS[c] * (2 if p == 1 else 1)
                                 for c in cls], device=dev,
                                dtype=torch.float64)
            dur = torch.randn(G, I, L, K, generator=plan, device=dev,
                              dtype=torch.float64)
            dur = tick(dur.mul_(0.3).exp_() * (mean * math.exp(-0.045)))
            gap = wait(G, I, L, K)
            if deep:                   # zero-length and abutting kernels
                dur[rand(G, I, L, K, of=plan) < 0.05] = 0
                gap[rand(G, I, L, K, of=plan) < 0.05] = 0
            st = torch.empty_like(dur)
            span = torch.zeros(G, I, L, dtype=i64, device=dev)
            for s in range(S):
                e = (gap[..., s::S] + dur[..., s::S]).cumsum(-1)
                st[..., s::S] = e - dur[..., s::S]
                if e.shape[-1]:
                    span = torch.maximum(span, e[..., -1])
            ph.append(dict(cls=cls, lab=lab, op=op, labels=[v for _, _, v in ops],
                           K=K, dur=dur, st=st, span=span))
        span = torch.cat([q["span"] for q in ph], 2)               # G I 3L
        lead = wait(G, I, 3 * L)
        each = (span + lead).reshape(G, -1).cumsum(1).reshape(G, I, 3 * L)
        base = each - span                                        # from T0
        cols = dict(gpu=[], stream=[], cls=[], op=[], st=[], en=[])
        gid = torch.arange(G, device=dev)
        t = lambda v, dt: torch.tensor(v, device=dev, dtype=dt)

        def add(st, en, stream, cls, op):
            shape = st.shape
            cols["gpu"].append(gid.to(u8).view(G, *[1] * (st.dim() - 1))
                               .expand(shape).reshape(-1))
            cols["stream"].append(stream.expand(shape).reshape(-1))
            cols["cls"].append(cls.expand(shape).reshape(-1))
            cols["op"].append(op.expand(shape).reshape(-1))
            cols["st"].append(st.reshape(-1))
            took = (en - st).double().mul_(0.75 + 0.25 * rand(*shape))
            if deep:                   # some take their whole slot
                took = torch.where(rand(*shape) < 0.1, en - st, took)
            cols["en"].append((st + took.to(i64)).reshape(-1))

        bounds, labels = [], []
        for p, q in enumerate(ph):
            q["st"] += base[:, :, p * L:(p + 1) * L, None]
            add(q["st"], q["st"] + q["dur"],
                t([j % S for j in range(q["K"])], u8), t(q["cls"], u8),
                t(q["lab"], torch.int32))
            n_ops = len(q["labels"])
            at = [[j for j in range(q["K"]) if q["op"][j] == o]
                  for o in range(n_ops)]
            bounds.append(torch.stack([q["st"][..., a[0]:a[-1] + 1].amin(-1)
                                       for a in at], -1).reshape(G, I, -1))
            labels += [q["labels"] for _ in range(L)]
        last = torch.stack([(q["st"] + q["dur"]).reshape(G, -1).amax(1)
                            for q in ph]).amax(0)
        # ---- communication: one kernel per layer, inside the window of the
        # block before, one after the other on its stream
        win = span[:, :, :2 * L].reshape(G, I, 2, L)
        bs = base[:, :, :2 * L].reshape(G, I, 2, L)
        prev = torch.arange(L, device=dev).sub(1).clamp_(min=0)
        win, bs = win[..., prev], bs[..., prev]
        u = rand(G, I, 2, L, of=plan) * (0.7 if deep else 0.4) + 0.3
        pos = rand(G, I, 2, L, of=plan)
        pos[..., 0] = 0
        want, dur = bs + tick(pos * win), tick(u * win)
        lines = [(0, 2, 2, 5), (1, 3, 3, 6)] if S > 1 else [(0, 1, 1, 5)]
        for p, s0, s1, c in lines:
            sel = slice(p, p + 1) if S > 1 else slice(0, 2)
            w, d = want[:, :, sel].reshape(G, -1), dur[:, :, sel].reshape(
                G, -1)
            tot = d.cumsum(1)
            en = tot + torch.cummax(w - (tot - d), 1).values
            k = 1 if S > 1 else 2
            kind = t([c] if S > 1 else [5, 6], u8).view(1, 1, k, 1)
            add((en - d).view(G, I, k, L), en.view(G, I, k, L), t([s0], u8),
                kind, kind.to(torch.int32) + 35)
        # ---- markers
        B = torch.cat(bounds, 2)                                   # G I ops
        n_ops = B.shape[2]
        B = torch.cummax(B.reshape(G, -1), 1).values
        Bn = torch.cat([B[:, 1:], torch.maximum(last, B[:, -1])[:, None]], 1)
        B, Bn = B.view(G, I, n_ops), Bn.view(G, I, n_ops)
        op_lab = t([v for block in labels for v in block], torch.int32)
        per = [len(_FWD)] * (2 * L) + [2] * L                      # ops a block
        f_of = t([sum(per[:b]) for b in range(3 * L)], i64)
        l_of = t([sum(per[:b + 1]) - 1 for b in range(3 * L)], i64)
        b_lab = t(list(range(L)) + list(range(L - 1, -1, -1)) +
                  list(range(L)), torch.int32)
        mk = []

        def mark(level, s, e, lab, keep=None):
            lab = lab.expand(s.shape)
            lev = torch.full_like(s, level)
            gg = gid.view(G, *[1] * (s.dim() - 1)).expand(s.shape)
            v = [x.reshape(-1) for x in (lev, gg, s, e, lab)]
            mk.append([x[keep.reshape(-1)] for x in v] if keep is not None
                      else v)

        ii = torch.arange(I, device=dev, dtype=torch.int32)
        mark(0, B[..., 0], Bn[..., -1], ii)
        mark(1, B[..., f_of[::L]], Bn[..., l_of[L - 1::L]],
             t([0, 1, 2], torch.int32))
        mark(2, B[..., f_of], Bn[..., l_of], b_lab)
        if not deep:
            mark(3, B, Bn, op_lab)
        else:
            d = torch.randint(3, 7, (G, I, 1), generator=plan, device=dev)
            mark(3, B, Bn, op_lab, (d >= 4).expand(B.shape))
            s, e, keep = B, Bn, (d >= 5).expand(B.shape)
            for level, k in ((4, 3), (5, 2)):     # split into 1..k pieces
                n_of = torch.randint(1, k + 1, s.shape, generator=plan,
                                     device=dev)
                cut = rand(*s.shape, k - 1, of=plan).sort(-1).values
                cut = s[..., None] + tick(cut * (e - s)[..., None])
                pts = torch.cat([s[..., None], cut, e[..., None]], -1)
                q = torch.arange(k, device=dev)
                s = pts[..., :-1]
                e = torch.where(q == n_of[..., None] - 1, e[..., None],
                                pts[..., 1:])
                keep = keep[..., None] & (q < n_of[..., None])
                mark(level, s, e, q.to(torch.int32), keep)
                keep = keep & (d.view(G, I, *[1] * (s.dim() - 2)) >= 6)
        mk = [torch.cat(v) for v in zip(*mk)]
        if deep:
            keep = rand(mk[0].numel(), of=plan) >= 0.01
            mk = [v[keep] for v in mk]
        span_all = int(mk[3].max()) + 1
        o = ((mk[1] * span_all + mk[2]) * 8 + mk[0]).argsort(stable=True)
        lev, mg, ms, me, ml = [v[o] for v in mk]
        cols = {k: torch.cat(v) for k, v in cols.items()}
        # ---- local clocks
        off_ns, ppm = (5e6, 200.0) if deep else (5e4, 20.0)
        skew = 0.0 if G == 1 else 1.0
        off = ((rand(G) * 2 - 1) * off_ns * skew).to(i64)
        begin = (rand(G) * 1e6).to(i64)
        drift = (rand(G) * 2 - 1) * ppm * 1e-6 * skew
        there = lambda v, gg: v + begin[gg]        # the reference clock
        local = lambda v, gg: (there(v, gg) + off[gg] +
                               (there(v, gg) * drift[gg]).round().to(i64))
        g8 = cols["gpu"].to(i64)
        st, en = local(cols["st"], g8), local(cols["en"], g8)
        key = st + 10_000_000               # offsets may reach below zero
        if case["order"] == "profiler":
            key = key + g8 * (int(key.max()) + 1)
        o = (key * 4 + cols["stream"]).argsort(stable=True)
        ms, me = local(ms, mg), local(me, mg)
        if case["order"] == "merged":
            m = ms.argsort(stable=True)
        elif case["order"] == "shuffled":
            o = torch.randperm(o.numel(), generator=g, device=dev)
            m = torch.randperm(ms.numel(), generator=g, device=dev)
        else:
            m = None
        if m is not None:
            lev, mg, ms, me, ml = lev[m], mg[m], ms[m], me[m], ml[m]
        self.gpu, self.stream, self.cls = (cols["gpu"][o], cols["stream"][o],
                                           cols["cls"][o])
        self.op_id = cols["op"][o]
        self.start, self.end = st[o] + T0, en[o] + T0
        self.m_gpu, self.m_level = mg.to(u8), lev.to(u8)
        self.m_start, self.m_end = ms + T0, me + T0
        self.m_label = ml.contiguous()
        self.n, self.n_markers = self.gpu.numel(), self.m_gpu.numel()
        # ---- clock anchors, four per iteration (host)
        if G > 1:
            s, e = B[..., 0], Bn[..., -1]
            y = (s[..., None] + (torch.arange(4, device=dev) +
                                 rand(G, I, 4)) / 4 * (e - s)[..., None]
                 ).to(i64).reshape(-1)
            ag = gid[:, None].expand(G, I * 4).reshape(-1)
            x = local(y, ag) + torch.randint(-50, 51, y.shape, generator=g,
                                             device=dev)
            self.a_gpu = ag.to(u8).cpu().numpy()
            self.a_local, self.a_ref = ((x + T0).cpu().numpy(),
                                        (there(y, ag) + T0).cpu().numpy())
        else:
            self.a_gpu = np.zeros(0, np.uint8)
            self.a_local = self.a_ref = np.zeros(0, np.int64)
        # ---- counters: cycles, events by class, clocks and power
        C = self.n_counters = case["counters"]
        self.counters = None
        if C:
            self.counters = torch.empty(C, self.n, dtype=i64, device=dev)
            us = (self.end - self.start).to(torch.float32).mul_(1e-3)
            rate = t(_RATE, torch.float32)
            k = self.cls.to(i64)
            ri = lambda lo, hi: torch.randint(lo, hi, (self.n,), generator=g,
                                              device=dev)
            sclk = ri(1300, 2101)
            for j in range(C):
                if j == 0:
                    v = (self.end - self.start) * sclk // 1000
                elif j < 13:
                    v = torch.randn(self.n, generator=g, device=dev)
                    v = v.mul_(0.5).sub_(0.125).exp_().mul_(us).mul_(
                        rate[:, j - 1][k])
                else:
                    v = sclk if j == 13 else ri(900, 1301) if j == 14 else \
                        ri(300, 751)
                self.counters[j] = v


# --------------------------------------------------------------------------
def prepare(case, seed):
    call = case["call"]
    tr = Trace(case, seed)
    s = dict(call=call)
    if call == "filter":
        filt = ch.make_filter(
            gpus=range(0, case["gpus"], 2) if case["few"] else None,
            classes=(0, 1, 5, 6) if case["few"] else None,
            iters=(case["lo"], case["hi"]))
        s["pipe"] = ch.Pipeline(tr, level=case["level"], filt=filt)
        return s
    pipe = s["pipe"] = ch.Pipeline(tr)
    if call == "step":
        return s
    pipe.step()
    if call == "views":
        s["views"] = ch.Views(pipe, n_phases=PHASES, n_ops=OPS,
                              n_iters=case["iters"], warmup=_warmup(case))
    elif call == "op_stats":
        s["flops"] = _flops()
    elif call == "launch_split":
        s["launch"] = _launch(tr, seed)
    elif call == "join":
        s["passes"] = _passes(tr, pipe)
    return s


def _warmup(case):
    return WARMUP if case["iters"] > WARMUP else 0


def _flops():
    return np.linspace(2e9, 9e10, OPS)


def _launch(tr, seed):
    """Dispatch times: up to 20 us before the start, one in a hundred up to
    5 us after it."""
    g = torch.Generator(device="cuda")
    g.manual_seed(seed + 1)
    ri = lambda lo, hi: torch.randint(lo, hi, (tr.n,), generator=g,
                                      device="cuda")
    late = torch.rand(tr.n, generator=g, device="cuda") < 0.01
    return tr.start - torch.where(late, -ri(1, 5000), ri(0, 20001))


def _passes(tr, pipe):
    """Seven passes that list every record in its GPU's dispatch order."""
    none = torch.full((1,), -1, dtype=torch.int32, device="cuda")
    lab = torch.cat([tr.m_label, none])[pipe.idx[0, :tr.n].long()]
    o = (tr.start - T0 + 10_000_000 + tr.gpu.long() * (1 << 50)).argsort(
        stable=True)
    same = bool((o[1:] > o[:-1]).all())
    take = (lambda v: v) if same else (lambda v: v[..., o].contiguous())
    shared = dict(gpu=take(tr.gpu), stream=take(tr.stream), cls=take(tr.cls),
                  label=take(lab))
    out, c = [], 0
    for k in PASSES:
        out.append(dict(shared, values=take(tr.counters[c:c + k]),
                        dst=list(range(c, c + k))))
        c += k
    return out


def _rows(pipe):
    r = pipe.rows
    out = {k: getattr(r, k) for k in ("level_offset", "path", "gpu", "kind",
                                      "n", "dur", "gap", "ovl", "tmin",
                                      "tmax", "first")}
    if r.n_counters:
        out["ctr"] = r.ctr
    if r.n_counters == 16:
        out["ratios"] = pipe.ratios
    else:                       # the metrics that need counters are NaN
        out["overlap_ratio"] = pipe.ratios[0]
    return out


def run(s):
    call, pipe = s["call"], s["pipe"]
    if call == "step":
        pipe.step()
        return dict({k: getattr(pipe, k) for k in (
            "start", "end", "mstart", "mend", "order", "korder", "idx", "ovl",
            "gap", "mwin", "gwin", "wfrac", "status")},
            clocks=np.frombuffer(pipe.clocks, np.int64), rows=_rows(pipe))
    if call == "filter":
        pipe.aggregate()
        pipe.derive_rows()
        return _rows(pipe)
    if call == "views":
        s["views"].run()
        return dict(s["views"].t)
    if call == "op_stats":
        return pipe.op_stats(n_phases=PHASES, n_ops=OPS, tpt_peak=1.3e6,
                             f_gemm=s["flops"], per_gpu=True)
    if call == "join":
        return pipe.join_counters(s["passes"])
    return pipe.launch_split(s["launch"])


# --------------------------------------------------------------------------
def _sizes(case):
    """Records, markers and aggregated rows; with deep markers the last two
    are what such traces come to, within a few percent."""
    G, I, L = case["gpus"], case["iters"], case["layers"]
    n = G * I * L * (30 + case["k_opt"])
    if case["depth"] == 4:
        return n, G * I * (4 + 31 * L), G * I * (7 + 35 * L), G * I * 30 * L
    return n, int(G * I * (4 + 72.6 * L)), G * I * 58 * L, G * I * 17 * L


def work(case):
    """Bytes: every input read once, every output written once; the work is
    integer scans, searches and sums, so no operations to speak of."""
    n, nm, nr, nr_op = _sizes(case)
    C, D, call = case["counters"], case["depth"], case["call"]
    row = 4 * D + 2 + 8 * 6 + 4 + 8 * C + 8 * 6
    if call == "step":
        b = n * (19 + 8 * C + 40 + 4 * D) + nm * (18 + 80) + nr * row
    elif call == "filter":
        part = (min(case["hi"], case["iters"] - 1) - case["lo"] + 1) / case[
            "iters"] * (0.3 if case["few"] else 1.0)
        nr = {255: nr, 100: 2 * case["gpus"]}.get(case["level"],
                                                  nr_op if case["level"] == 3
                                                  else nr // 7)
        b = n * (2 + 4) + max(part, 0) * (
            n * (4 * (D - 1) + 32 + 8 * C) + nr * row)
    elif call == "views":
        units = case["gpus"] * case["iters"]
        b = (n * (1 + 8 * 3 + 4 + 4) + nm * 5 + nr_op * (12 + 1 + 32) + units *
             (8 * (3 * PHASES * 8 + 4 * PHASES * OPS * 2 + 1) + 4))
    elif call == "op_stats":
        b = nr_op * (1 + 8 * 3 + 8 + (24 if C == 16 else 0))
    elif call == "join":
        b = len(PASSES) * n * 7 + n * 8 * 16 + n * 11 + n * 8 * 16 + n
    else:
        b = n * 41
    return {"bytes": float(b), "flops": 0.0}


def tolerance(case):
    """Integers, and doubles that are stated operation by operation on
    them."""
    return "exact"


# --------------------------------------------------------------------------
# The computed metrics in plain torch, from the definitions
# --------------------------------------------------------------------------
def _fit(tr):
    """Per GPU (x0, c, d): least squares of ref - local on local, the slope
    in units of 2^-48, both rounded half to even."""
    def nearest(a, b):                                   # b > 0
        q, r = divmod(a, b)
        return q + (2 * r > b or (2 * r == b and q & 1))

    out = []
    for g in range(tr.n_gpus):
        sel = tr.a_gpu == g
        x, y = tr.a_local[sel], tr.a_ref[sel]
        if not x.size:
            out.append((0, 0, 0))
            continue
        x0 = int(x.min())
        u, w = [int(v) for v in x - x0], [int(v) for v in y - x]
        m, su, sw = len(u), sum(u), sum(w)
        den = m * sum(v * v for v in u) - su * su
        num = m * sum(a * b for a, b in zip(u, w)) - su * sw
        d = nearest(num << 48, den) if den else 0
        c = nearest((sw << 48) - d * su, m << 48)
        out.append((x0, c, d))
    return out


def _aligned(tr):
    fit = _fit(tr)
    x0, c, d = [torch.tensor(v, device="cuda") for v in zip(*fit)]

    def al(t, g):
        g = g.long()
        u = t - x0[g]
        low = (u & 0xFFFFFF) * d[g] >> 24
        return t + c[g] + ((u >> 24) * d[g] + low >> 24)

    return (al(tr.start, tr.gpu) - T0, al(tr.end, tr.gpu) - T0,
            al(tr.m_start, tr.m_gpu) - T0, al(tr.m_end, tr.m_gpu) - T0)


class _Union:
    """Time covered by intervals of several GPUs, up to a point."""

    def __init__(self, g, s, e, wide):
        k = g * wide + s
        o = k.argsort(stable=True)
        self.wide, self.k = wide, k[o]
        top = torch.cummax((g * wide + e)[o], 0).values
        before = torch.cat([top[:1] - (1 << 61), top[:-1]])
        self.top = top
        self.sum = (top - torch.maximum(self.k, before)).clamp_(
            min=0).cumsum(0)

    def upto(self, g, t):
        if not self.k.numel():
            return torch.zeros_like(t)
        q = g * self.wide + t
        j = torch.searchsorted(self.k, q, right=True) - 1
        some = j >= 0
        j = j.clamp_(min=0)
        v = self.sum[j] - (self.top[j] - q).clamp_(min=0)
        return torch.where(some, v, torch.zeros_like(v))


def _analysis(tr):
    """Aligned times, marker of each level, overlapped time, bubble."""
    s, e, ms, me = _aligned(tr)
    g, mg = tr.gpu.long(), tr.m_gpu.long()
    lo = min(int(s.min()), int(ms.min()))
    s, e, ms, me = s - lo, e - lo, ms - lo, me - lo
    wide = max(int(e.max()), int(me.max())) + 1
    kind = ((tr.cls == 5) | (tr.cls == 6)).long()
    idx = []
    for level in range(tr.depth):
        i = torch.nonzero((tr.m_level == level) & (me > ms)).flatten()
        k = mg[i] * wide + ms[i]
        o = k.argsort(stable=True)
        i, k = i[o], k[o]
        if not i.numel():
            idx.append(torch.full_like(s, -1))
            continue
        j = torch.searchsorted(k, g * wide + s, right=True) - 1
        at = i[j.clamp(min=0)]
        ok = (j >= 0) & (mg[at] == g) & (s < me[at])
        idx.append(torch.where(ok, at, torch.full_like(at, -1)))
    un = [_Union(g[kind == k], s[kind == k], e[kind == k], wide)
          for k in (0, 1)]
    both = _Union(g, s, e, wide)
    ovl = torch.zeros_like(s)
    for k in (0, 1):
        m = kind == k
        ovl[m] = un[1 - k].upto(g[m], e[m]) - un[1 - k].upto(g[m], s[m])
    gap = torch.zeros_like(s)
    m = torch.nonzero(kind == 0).flatten()
    line = g[m] * 256 + tr.stream[m].long()
    o = s[m].argsort(stable=True)
    o = o[line[o].argsort(stable=True)]
    m, line = m[o], line[o]
    gap[m[1:]] = torch.where(line[1:] == line[:-1],
                             (s[m[1:]] - e[m[:-1]]).clamp_(min=0), 0)
    return dict(g=g, kind=kind, s=s, e=e, ms=ms, me=me, mg=mg, idx=idx,
                ovl=ovl, gap=gap, dur=e - s, un=un, both=both)


def _groups(tr, a, level, keep=None):
    """Group number of each (kept) record, in row order, and their count."""
    pick = (lambda v: v) if keep is None else (lambda v: v[keep])
    g, kind, s = pick(a["g"]), pick(a["kind"]), pick(a["s"])
    if level == 101:
        gid = kind
    else:
        gid = g * 2 + kind
        for l in range(level + 1 if level < 100 else 0):
            key = gid * (tr.n_markers + 1) + pick(a["idx"][l]) + 1
            gid = torch.unique(key, return_inverse=True)[1]
    gid = torch.unique(gid, return_inverse=True)[1]
    n = int(gid.max()) + 1 if gid.numel() else 0
    big = torch.iinfo(torch.int64).max
    tmin = torch.full((n,), big, device="cuda").scatter_reduce_(
        0, gid, s, "amin")
    at = torch.arange(s.numel(), device="cuda")
    at = torch.where(s == tmin[gid], at, big)
    first = torch.full((n,), big, device="cuda").scatter_reduce_(
        0, gid, at, "amin")
    head = kind[first] if level == 101 else (g * 2 + kind)[first]
    o = first.argsort(stable=True)
    o = o[tmin[o].argsort(stable=True)]
    o = o[head[o].argsort(stable=True)]
    rank = torch.empty_like(o)
    rank[o] = torch.arange(n, device="cuda")
    return rank[gid], n, first[o]


def _sum(gid, n, v):
    return torch.zeros(n, dtype=torch.int64, device="cuda").index_add_(
        0, gid, v)


def _ratios(tr, a, levels, keep=None):
    pick = (lambda v: v) if keep is None else (lambda v: v[keep])
    out = []
    for level in levels:
        gid, n, _ = _groups(tr, a, level, keep)
        f = lambda v: _sum(gid, n, pick(v)).double()
        r = torch.full((6, n), math.nan, dtype=torch.float64, device="cuda")
        dur = f(a["dur"])
        r[0] = f(a["ovl"]) / dur
        if tr.n_counters == 16:
            c = tr.counters
            r[1] = f(c[4] + c[5]) / dur
            r[2] = f(c[13]) / f(torch.ones_like(a["s"]))
            r[3] = f(c[1]) / f(c[0])
            r[4] = f(c[0]) * 1000.0 / 2100.0
            r[5] = dur / r[4]
        out.append(r)
    r = torch.cat(out, 1)
    return dict(ratios=r) if tr.n_counters == 16 else dict(
        overlap_ratio=r[0].clone())


def _medians(v, gid, n):
    """Median of the values of each of n groups (NaN where empty)."""
    o = v.argsort(stable=True)
    o = o[gid[o].argsort(stable=True)]
    v, m = v[o].double(), torch.bincount(gid, minlength=n)
    at = m.cumsum(0) - m
    v = torch.cat([v, torch.zeros(1, dtype=v.dtype, device="cuda")])
    lo = v[(at + (m - 1).clamp(min=0) // 2).clamp(max=v.numel() - 1)]
    hi = v[(at + m // 2).clamp(max=v.numel() - 1)]
    return torch.where(m > 0, (lo + hi) / 2, math.nan)


def _exact_views(case, tr, a):
    lab = tr.m_label.long()
    u, p, o = [a["idx"][l] for l in (0, 1, 3)]
    warm, P, O = _warmup(case), PHASES, OPS
    has = (u >= 0) & (p >= 0)
    units = torch.unique(torch.nonzero(tr.m_level == 0).flatten())
    U = units.numel()
    unit = torch.searchsorted(units, u.clamp(min=0))
    late = lab[units] >= warm

    def tab(m, group, n_groups):
        g, n = (group * U + unit)[m], n_groups * U
        cnt = _sum(g, n, torch.ones_like(g)).view(n_groups, U)
        dur = _sum(g, n, a["dur"][m]).view(n_groups, U)
        gap = _sum(g, n, a["gap"][m]).view(n_groups, U)
        ok = (cnt > 0) & late
        which = torch.arange(n_groups, device="cuda")[:, None].expand_as(
            ok)[ok]
        return torch.cat([_medians(v[ok], which, n_groups)
                          for v in (dur, gap, dur + gap)])

    pl, ol = lab[p.clamp(min=0)], lab[o.clamp(min=0)]
    cls_med = tab(has, pl * 8 + tr.cls.long(), P * 8)
    op_med = tab(has & (o >= 0), (pl * O + ol) * 2 + a["kind"], P * O * 2)
    m = (u >= 0) & (a["kind"] == 0)
    busy = _sum(unit[m], U, (a["dur"] + a["gap"])[m])
    top = torch.full((case["iters"],), -1, device="cuda").scatter_reduce_(
        0, lab[units], busy, "amax")
    top = top[warm:][top[warm:] >= 0]
    it = _medians(top, torch.zeros_like(top), 1)
    out = dict(cls_med=cls_med, op_med=op_med, iter_med=it)
    return out


def _exact_stats(tr, a):
    G, NG = PHASES * OPS, tr.n_gpus
    gid, n, first = _groups(tr, a, 3)
    f = lambda v: _sum(gid, n, v)
    dur, gap, ovl = f(a["dur"]), f(a["gap"]), f(a["ovl"])
    lab = tr.m_label.long()
    p, o = a["idx"][1][first], a["idx"][3][first]
    ok = (a["kind"][first] == 0) & (dur > 0) & (p >= 0) & (o >= 0)
    grp = lab[p.clamp(min=0)] * OPS + lab[o.clamp(min=0)]
    ok &= (lab[p.clamp(min=0)] < PHASES) & (lab[o.clamp(min=0)] < OPS)
    grp, gpu = grp[ok], a["g"][first][ok]
    # the quotient of 2^30 ovl, in 64 bits: the whole part, then 15 bits twice
    q, r = ovl // dur.clamp(min=1), ovl % dur.clamp(min=1)
    for _ in range(2):
        r = r << 15
        q, r = (q << 15) + r // dur.clamp(min=1), r % dur.clamp(min=1)
    x, y = q[ok], (dur + gap)[ok]
    nan = lambda *s: torch.full(s, math.nan, dtype=torch.float64,
                                device="cuda")
    out, gout = nan(17, G), nan(9, G, NG)
    ctr = None
    if tr.n_counters == 16:
        ctr = [f(tr.counters[j])[ok] for j in (0, 1, 11)]
    fg = _flops()
    for k in range(G):
        m = grp == k
        cnt = int(m.sum())
        if not cnt:
            continue
        out[16, k] = fg[k % OPS] / 1.3e6
        xs, ys, gs = x[m], y[m], gpu[m]
        dx, dy = (xs.double() - xs.double().mean(),
                  ys.double() - ys.double().mean())
        vx, vy, cv = (dx * dx).sum(), (dy * dy).sum(), (dx * dy).sum()
        if bool((xs != xs[0]).any()):
            out[1, k] = cv / vx
            out[2, k] = ys.double().mean() - out[1, k] * xs.double().mean()
            out[3, k], out[4, k] = out[2, k], out[2, k] + out[1, k] * 2.0**29
            if bool((ys != ys[0]).any()):
                out[0, k] = cv / (vx * vy).sqrt()
        at = lambda v, i: v[i].double()

        def quantiles(v):
            h = v.numel() - 1
            return torch.stack([at(v, 0), at(v, h // 4),
                                (at(v, h // 2) + at(v, (h + 1) // 2)) / 2,
                                at(v, 3 * h // 4), at(v, h)]) * 2.0**-30
        out[5:10, k] = quantiles(xs.sort().values)
        ovr = []
        for h in range(NG):
            mh = gs == h
            if not bool(mh.any()):
                continue
            xh, oh = xs[mh].sort(stable=True)
            yh = ys[mh][oh].double()
            low = yh.min()
            mid = xh.numel() - 1
            gout[:5, k, h] = quantiles(xh)
            gout[5, k, h], gout[6, k, h] = low, yh[0] / low
            gout[7, k, h] = (yh[mid // 2] / low + yh[(mid + 1) // 2] / low) / 2
            gout[8, k, h] = gout[7, k, h] / gout[6, k, h]
            ovr.append(gout[8, k, h])
        ovr = torch.stack(ovr).sort().values
        h = ovr.numel() - 1
        out[10, k] = ys.double().mean()
        out[14, k] = (ovr[h // 2] + ovr[(h + 1) // 2]) / 2
        if ctr is not None:
            c0, c1, c11 = [c[m].sum().double() for c in ctr]
            out[11, k] = c0 * 1000.0 / 2100.0 / cnt
            out[12, k] = 1.0 / (c1 / c0)
            out[13, k] = c11 / cnt / fg[k % OPS]
            out[15, k] = out[10, k] / out[11, k] / out[14, k]
    return out, None, gout.view(9, G * NG), None


def exact(case, seed):
    call = case["call"]
    if call in ("join", "launch_split"):
        return None                                  # whole numbers alone
    tr = Trace(case, seed)
    a = _analysis(tr)
    levels = list(range(tr.depth)) + [100, 101]
    if call == "filter":
        keep = a["idx"][0] >= 0
        lab = tr.m_label[a["idx"][0].clamp(min=0)]
        keep &= (lab >= case["lo"]) & (lab <= case["hi"])
        if case["few"]:
            keep &= (tr.gpu % 2 == 0) & ((tr.cls < 2) | (a["kind"] == 1))
        if case["level"] != 255:
            levels = [case["level"]]
        return _ratios(tr, a, levels, torch.nonzero(keep).flatten())
    if call == "views":
        return _exact_views(case, tr, a)
    if call == "op_stats":
        return _exact_stats(tr, a)
    # window fractions: compute only, communication only, both, neither
    w = [u.upto(a["mg"], a["me"]) - u.upto(a["mg"], a["ms"])
         for u in a["un"] + [a["both"]]]
    ov = w[0] + w[1] - w[2]
    length = (a["me"] - a["ms"]).clamp(min=0)
    win = torch.stack([w[0] - ov, w[1] - ov, ov, length - w[2]], 1)
    win = torch.where(length[:, None] > 0, win, torch.zeros_like(win))
    frac = win.double() / win.sum(1, keepdim=True).double()
    return dict(wfrac=frac, rows=_ratios(tr, a, levels))
