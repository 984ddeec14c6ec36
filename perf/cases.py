"""Performance cases of the wave propagator: the runs its users make.

Each case is one pass through the public entry points of
``paper_2204_03775_amd.wave``, as a user's program calls them.  The kinds are

``steps``     a driver that owns the time loop: one ``step`` call per time step;
``shot``      a whole shot with ``run`` (optionally replayed from a HIP graph),
              traces and the final field as results;
``monitor``   a shot run in segments, with the field exported and the watchdog
              asked after each (snapshots of a long run);
``gradient``  an inversion iteration on a kept propagator: checkpointed forward
              run, misfit, adjoint run to velocity;
``autograd``  the same through ``traces_of_velocity`` and ``torch.autograd``;
``batch``     many uneven shots advanced together.

The models are layered media with smooth noise, with a Ricker point source, a
line of receivers and an absorbing sponge, as the workloads of
``paper_2204_03775_amd.inputs``, made on the GPU from the seed alone.
"""
import math
import random

import torch

from paper_2204_03775_amd import inputs, wave

H = (10.0, 10.0, 10.0)
DT = inputs.cfl_dt(4500.0, 10.0, 0.8)
FREQ = 12.0
# bytes per cell and step that a storage form moves: every field read once, the
# new level (and the step change) written once
STEP_BYTES = {"f32": 16, "f16": 8, "bf16": 8, "f16uv": 10, "bf16uv": 10}
STEP_FLOPS = 51     # per cell and step, the paper's convention
ADJOINT_BYTES = 36  # phi twice, k, the forward level and the FP64 sum read; phi and the sum written
ADJOINT_FLOPS = 100


def _shot(name, dtype, nx, ny, nz, nt, graph=False):
    return {"name": name, "kind": "shot", "dtype": dtype, "nx": nx, "ny": ny, "nz": nz, "nt": nt, "graph": graph}


def listed():
    return [
        # the smallest calls: a small ragged model stepped by the caller, one call per step
        {"name": "steps_37x21x19", "kind": "steps", "dtype": "f32", "nx": 37, "ny": 21, "nz": 19, "nt": 30},
        # the parity shot's size, bound by launches: replayed from a graph
        _shot("shot_64_graph", "f32", 64, 64, 64, 100, True),
        # snapshots and watchdog of a reduced-precision run (the 128^3 crop's size)
        {"name": "monitor_128_f16uv", "kind": "monitor", "dtype": "f16uv", "nx": 128, "ny": 128, "nz": 128,
         "nt": 200, "segments": 4},
        # a medium shot, whose fields fit in the memory-side cache
        _shot("shot_256_f32", "f32", 256, 256, 256, 200),
        # the benchmark shot's grid
        _shot("shot_512_f32", "f32", 512, 512, 512, 200),
        # the paper's plane (Table 3), ragged in x and y
        _shot("shot_755x994x200_f32", "f32", 755, 994, 200, 50),
        # the benchmark grid in the 16-bit form that meets the accuracy bound
        _shot("shot_512_f16uv", "f16uv", 512, 512, 512, 200),
        # the BF16 form on a ragged grid near the paper's 400 x 400 plane
        _shot("shot_401x397x300_bf16uv", "bf16uv", 401, 397, 300, 150),
        # two-level 16-bit storage at a production shot's size
        _shot("shot_320x288x272_f16", "f16", 320, 288, 272, 150),
        # an inversion iteration on the gradient shot's grid, every level kept
        {"name": "gradient_256", "kind": "gradient", "nx": 256, "ny": 256, "nz": 256, "nt": 150, "every": 0},
        # the same through autograd on a ragged grid with checkpoints
        {"name": "autograd_203x181x157", "kind": "autograd", "nx": 203, "ny": 181, "nz": 157, "nt": 120,
         "every": 25},
        # a survey's uneven shots, each with its own kernel on concurrent streams
        {"name": "batch_16_uneven", "kind": "batch", "shots": 16, "lo": 96, "hi": 320, "sizes": 2207, "nt": 60,
         "schedule": 1, "nstreams": 4},
    ]


def _size(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _grid(rng, lo, hi, most):
    while True:
        n = [_size(rng, lo, hi) for _ in range(3)]
        if n[0] * n[1] * n[2] <= most:
            return {"nx": n[0], "ny": n[1], "nz": n[2]}


def draw(rng):
    kind = rng.choice(("steps", "shot", "shot", "shot", "shot16", "shot16", "shot16", "monitor", "gradient",
                       "autograd", "batch", "batch"))
    if kind == "steps":
        return {"kind": "steps", "dtype": "f32", **_grid(rng, 17, 96, 1 << 20), "nt": rng.randint(20, 60)}
    if kind in ("shot", "shot16"):
        dtype = "f32" if kind == "shot" else rng.choice(("f16uv", "bf16uv", "f16", "bf16"))
        g = _grid(rng, 48, 760, 1 << 27)
        cells = g["nx"] * g["ny"] * g["nz"]
        nt = min(_size(rng, 40, 400), max(20, int(2.6e10 / cells)))
        return {"kind": "shot", "dtype": dtype, **g, "nt": nt, "graph": cells < (1 << 22) and rng.random() < 0.5}
    if kind == "monitor":
        return {"kind": "monitor", "dtype": rng.choice(("f32", "f16uv", "bf16uv")), **_grid(rng, 64, 320, 1 << 24),
                "nt": 40 * rng.randint(2, 5), "segments": rng.randint(2, 5)}
    if kind in ("gradient", "autograd"):
        g = _grid(rng, 48, 320, 1 << 24)
        return {"kind": kind, **g, "nt": rng.randint(60, 140), "every": rng.choice((0, 0, 25, 40))}
    small = rng.random() < 0.5
    return {"kind": "batch", "shots": rng.randint(6, 20), "lo": 32 if small else 96, "hi": 96 if small else 256,
            "sizes": rng.randint(1, 1 << 20), "nt": rng.randint(30, 60), "schedule": 0 if small else rng.choice((0, 1)),
            "nstreams": rng.choice((2, 4))}


# --- inputs -------------------------------------------------------------------


def _device():
    return torch.device("cuda" if torch.cuda.is_available() else "cpu")


def _model(shape, seed):
    """Layered velocity (3..6 layers, 1500..4500 m/s) with 5 % smooth noise."""
    dev = _device()
    r = random.Random(seed)
    g = torch.Generator(device=dev)
    g.manual_seed(seed)
    nz = shape[0]
    vel = sorted(r.uniform(1500.0, 4200.0) for _ in range(r.randint(3, 6)))
    layer = (torch.arange(nz, device=dev) * len(vel)) // nz
    v = torch.tensor(vel, device=dev)[layer][:, None, None]
    coarse = torch.rand([1, 1] + [n // 6 + 2 for n in shape], generator=g, device=dev) * 2.0 - 1.0
    noise = torch.nn.functional.interpolate(coarse, size=shape, mode="trilinear", align_corners=True)[0, 0]
    return (v * (1.0 + 0.05 * noise)).contiguous()


class _Input:
    """Everything of one shot: model, source, receivers and sponge."""

    def __init__(self, nx, ny, nz, nt, seed, most_rec=256):
        r = random.Random(seed * 7 + 1)
        self.shape, self.nt = (nz, ny, nx), nt
        self.v = _model(self.shape, seed)
        self.k = ((self.v.double() * DT) ** 2).float()
        self.width = min(20, min(self.shape) // 6)
        self.alpha = 0.015 * 20.0 / max(self.width, 1) if self.width < 20 else 0.015
        # a surface survey: the source a few cells below the line of receivers
        m = self.width + 2
        z, y = min(nz - 1, m), ny // 2
        self.src = (min(nz - 1, z + r.randint(2, 4)), min(ny - 1, y + r.randint(0, 2)), r.randint(m, nx - 1 - m))
        w = inputs.ricker(FREQ * 2.0 if nt < 100 else FREQ, nt, DT)
        self.wavelet = w
        v_src = float(self.v[self.src])
        s = torch.tensor(inputs.point_source_values(w, v_src, DT, H))
        # of order one per step, as traces are usually scaled
        self.s = (s / s.abs().max()).to(torch.float32).to(self.v.device)
        nrec = min(most_rec, nx - 2 * m)
        self.rec = [[z, y, m + (i * (nx - 1 - 2 * m)) // max(nrec - 1, 1)] for i in range(nrec)]

    def propagator(self, dtype, stream=None):
        nz, ny, nx = self.shape
        p = wave.Propagator(nx, ny, nz, H, self.k, src=self.src, rec=self.rec, sponge_width=self.width,
                            sponge_alpha=self.alpha, stream=stream, dtype=dtype)
        p.record(self.nt)
        return p

    def observed(self):
        """Traces of the first arrivals in a constant 2500 m/s medium, [nt][nrec]."""
        dev = self.v.device
        d = torch.tensor([[abs(a - b) * 10.0 for a, b in zip(self.src, r)] for r in self.rec], device=dev)
        dist = d.square().sum(1).sqrt().clamp(min=10.0)
        t = torch.arange(self.nt, device=dev, dtype=torch.float32)[:, None] * DT - dist[None, :] / 2500.0
        a = (math.pi * FREQ * (t - 1.0 / FREQ)) ** 2
        return ((1.0 - 2.0 * a) * torch.exp(-a) * (30.0 / dist)[None, :]).contiguous()


def _batch_sizes(case):
    r = random.Random(case["sizes"])
    dim = lambda: r.randint(case["lo"], case["hi"])  # noqa: E731
    return [(dim(), dim(), min(dim(), 256)) for _ in range(case["shots"])]


def _batch_inputs(case, seed):
    return [_Input(*n, case["nt"], seed * 64 + i, 128) for i, n in enumerate(_batch_sizes(case))]


class _State:
    pass


def prepare(case, seed):
    st = _State()
    st.case = case
    kind = case["kind"]
    if kind == "batch":
        ins = _batch_inputs(case, seed)
        st.stream = torch.cuda.Stream()
        st.stream.wait_stream(torch.cuda.current_stream())
        st.props = [i.propagator("f32", st.stream) for i in ins]
        st.srcs = [i.s for i in ins]
        st.batch = wave.Batch(st.props, stream=st.stream, use_graph=True)
        st.batch.set_schedule(case["schedule"], case["nstreams"])
        return st
    inp = _Input(case["nx"], case["ny"], case["nz"], case["nt"], seed)
    if kind == "autograd":
        st.v, st.observed = inp.v, inp.observed()
        st.survey = wave.Survey(H, DT, inp.nt, inp.src, inp.s, inp.rec, inp.width, inp.alpha, every=case["every"])
        return st
    st.src = inp.s
    if kind == "steps":
        st.values = inp.s.tolist()
    if case.get("graph"):
        st.stream = torch.cuda.Stream()
        st.stream.wait_stream(torch.cuda.current_stream())
        st.prop = inp.propagator(case["dtype"], st.stream)
        st.prop.use_graph()
    else:
        st.prop = inp.propagator(case.get("dtype", "f32"))
    if kind == "gradient":
        st.v, st.observed = inp.v, inp.observed()
    return st


# --- passes -------------------------------------------------------------------


def _field(prop):
    return prop.interior(prop.fields()[0]) if prop.dtype == wave.WAVE_F32 else prop.export(0)


def _run_shot(st):
    p = st.prop
    p.reset()
    p.run(st.case["nt"], st.src)
    return {"u": _field(p), "traces": p.traces[:, :p.nrec]}


def run(state):
    case, kind = state.case, state.case["kind"]
    if kind == "steps":
        p = state.prop
        p.reset()
        for s in state.values:
            p.step(s)
        return {"u": _field(p), "traces": p.traces[:, :p.nrec]}
    if kind == "shot":
        if not case.get("graph"):
            return _run_shot(state)
        cur = torch.cuda.current_stream()
        state.stream.wait_stream(cur)
        with torch.cuda.stream(state.stream):
            out = _run_shot(state)
        cur.wait_stream(state.stream)
        return out
    if kind == "monitor":
        p, per = state.prop, case["nt"] // case["segments"]
        p.reset()
        out = {"snapshots": [], "nonfinite": []}
        for i in range(case["segments"]):
            p.run(per, state.src[i * per:(i + 1) * per])
            out["snapshots"].append(p.export(0))
            out["nonfinite"].append(sum(p.check()))
        out["traces"] = p.traces[:per * case["segments"], :p.nrec]
        return out
    if kind == "gradient":
        p = state.prop
        p.reset()
        p.forward_checkpointed(case["nt"], state.src, case["every"])
        misfit, residual = wave.misfit(p.traces, state.observed)
        grad = p.adjoint_velocity(residual, state.v, DT)
        return {"misfit": misfit, "traces": p.traces, "grad": grad}
    if kind == "autograd":
        v = state.v.detach().requires_grad_()
        traces = wave.traces_of_velocity(v, state.survey)
        loss = 0.5 * (traces - state.observed).double().square().sum()
        loss.backward()
        return {"misfit": loss.detach(), "traces": traces.detach(), "grad": v.grad}
    for p in state.props:
        p.reset()
    state.batch.run(case["nt"], state.srcs)
    return [{"u": _field(p), "traces": p.traces[:, :p.nrec]} for p in state.props]


def work(case):
    if case["kind"] == "batch":
        n = sum(a * b * c for a, b, c in _batch_sizes(case)) * case["nt"]
        return {"bytes": n * STEP_BYTES["f32"], "flops": n * STEP_FLOPS}
    cells = case["nx"] * case["ny"] * case["nz"]
    n = cells * case["nt"]
    b, f = n * STEP_BYTES[case.get("dtype", "f32")], n * STEP_FLOPS
    if case["kind"] in ("gradient", "autograd"):
        b, f = b + n * ADJOINT_BYTES, f + n * ADJOINT_FLOPS
    if case["kind"] == "monitor":
        b += case["segments"] * cells * (4 + (4 if case["dtype"] == "f32" else 2))
    return {"bytes": b, "flops": f}


# --- the same in 64 bits ------------------------------------------------------

WEIGHTS = (-205.0 / 72.0, 8.0 / 5.0, -1.0 / 5.0, 8.0 / 315.0, -1.0 / 560.0)


class _Exact:
    """The scheme of a shot in FP64 with plain tensor operations."""

    def __init__(self, inp):
        self.inp, self.dev = inp, inp.v.device
        self.k = inp.k.double()
        prof = []
        for n in inp.shape:
            d = torch.minimum(torch.arange(n), n - 1 - torch.arange(n)).double()
            g = torch.exp(-(inp.alpha * (inp.width - d)) ** 2)
            prof.append(torch.where(d < inp.width, g, torch.ones_like(g)).to(self.dev))
        self.g = prof[0][:, None, None] * prof[1][None, :, None] * prof[2][None, None, :]
        self.s = inp.s.double()
        rec = torch.tensor(inp.rec, device=self.dev)
        self.at = (rec[:, 0], rec[:, 1], rec[:, 2])

    def padded(self):
        return torch.zeros([n + 8 for n in self.inp.shape], dtype=torch.float64, device=self.dev)

    @staticmethod
    def inner(p):
        return p[4:-4, 4:-4, 4:-4]

    def lap(self, p):
        n = self.inp.shape
        out = self.inner(p) * (WEIGHTS[0] * sum(1.0 / h ** 2 for h in H))
        for axis, h in ((0, H[2]), (1, H[1]), (2, H[0])):
            for m in range(1, 5):
                for o in (4 - m, 4 + m):
                    lo = [4, 4, 4]
                    lo[axis] = o
                    out.add_(p[tuple(slice(a, a + b) for a, b in zip(lo, n))], alpha=WEIGHTS[m] / h ** 2)
        return out

    def forward(self, nt, keep=None, at_steps=()):
        cur, prev = self.padded(), self.padded()
        traces, snaps = [], []
        for n in range(nt):
            lap = self.lap(cur)
            if keep is not None:
                keep.append(lap)
                lap = lap.clone()
            u = self.inner(prev)
            u.mul_(self.g).neg_().add_(lap.mul_(self.k)).add_(self.inner(cur), alpha=2.0).mul_(self.g)
            u[self.inp.src] += self.s[n]
            cur, prev = prev, cur
            traces.append(u[self.at])
            if n + 1 in at_steps:
                snaps.append(self.inner(cur).clone())
        return self.inner(cur), torch.stack(traces), snaps

    def adjoint(self, laps, g):
        """dJ/dk for dJ/d traces = g, given the Laplacians of the forward levels."""
        one, two, arg = (self.padded() for _ in range(3))
        grad = torch.zeros(self.inp.shape, dtype=torch.float64, device=self.dev)
        for m in range(len(laps), 0, -1):
            l1, l2 = self.inner(one), self.inner(two)
            torch.mul(l1, self.g, out=self.inner(arg))
            new = self.inner(arg) * 2.0 - l2 * self.g ** 2
            self.inner(arg).mul_(self.k)
            new += self.lap(arg)
            new.index_put_(self.at, g[m - 1], accumulate=True)
            l2.copy_(new)
            one, two = two, one
            grad += new * self.g * laps[m - 1]
        return grad


def exact(case, seed):
    kind = case["kind"]
    if kind == "batch":
        out = []
        for inp in _batch_inputs(case, seed):
            u, traces, _ = _Exact(inp).forward(case["nt"])
            out.append({"u": u, "traces": traces})
        return out
    if case.get("dtype") == "bf16":
        return None  # two levels of 8 significant bits: the stored values are not near the FP64 ones
    inp = _Input(case["nx"], case["ny"], case["nz"], case["nt"], seed)
    e = _Exact(inp)
    if kind in ("steps", "shot"):
        u, traces, _ = e.forward(case["nt"])
        return {"u": u, "traces": traces}
    if kind == "monitor":
        per, parts = case["nt"] // case["segments"], case["segments"]
        _, traces, snaps = e.forward(per * parts, at_steps=[per * (i + 1) for i in range(parts)])
        return {"snapshots": snaps, "nonfinite": [None] * parts, "traces": traces}
    laps = []
    _, traces, _ = e.forward(case["nt"], keep=laps)
    r = traces - inp.observed().double()
    grad = e.adjoint(laps, r) * (2.0 * DT * DT) * inp.v.double()
    return {"misfit": 0.5 * r.square().sum(), "traces": traces, "grad": grad}
