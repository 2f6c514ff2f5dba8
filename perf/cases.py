"""The work this library is used for, as cases that can be timed and compared.

Every case goes through the public binding (`paper_1902_04610_amd.salus`): a pool over a device
buffer, one job per lane, and per pass what a serving or tuning program does - give the jobs work,
schedule a round, launch it.  Kinds:

  forward   one packed inference round (schedule + grouped_forward or grouped_forward_static)
  train     one packed training step (schedule + grouped_train_step)
  compact   a job leaves, the persistent region is compacted, a new job of the same size arrives
  switch    a job's persistent state leaves to pinned host memory and comes back

A case holds plain values only; row counts of a mixed round are drawn from the case's own `mix`
number, so that `work` knows them, and the data come from `prepare`'s seed.
"""
import ctypes

import numpy as np
import torch

from paper_1902_04610_amd import salus

_MLP = "1024-4096-1024-1024"          # the inference models of the packing benchmark
_TUNE = "2048-2048-2048-2048-1000"    # the training jobs of the tuning benchmark


def _fwd(name, jobs, dims, rows, dtype="bf16", act="gelu", layout="rows", mix=1, static=False):
    """rows: "7" every job has 7, "1..32" drawn per job (log-uniform), "poisson" request arrivals."""
    c = dict(kind="forward", jobs=jobs, dims=dims, rows=rows, dtype=dtype, act=act, layout=layout, mix=mix, static=static)
    return dict(c, name=name) if name else c


def _train(name, jobs, dims, rows):
    c = dict(kind="train", jobs=jobs, dims=dims, rows=rows)
    return dict(c, name=name) if name else c


def listed():
    return [
        # the smallest round: two float jobs of two 256 x 256 layers, 8 rows; launches and host work
        _fwd("float_2x256_b8", 2, "256-256-256", "8", dtype="f32", act="relu"),
        # float models kept in full precision, widths that are no multiple of a tile, ordinary batches
        _fwd("float_12_ragged", 12, "516-1204-780-388", "1..128", dtype="f32", mix=3),
        # one model, one request, the entry point of latency-bound serving loops
        _fwd("serve_one_request", 1, _MLP, "1", layout="strip", static=True),
        # the packing benchmark's round: 64 resident models, Poisson arrivals, 1 - 32 rows each
        _fwd("packing_poisson", 64, _MLP, "poisson", layout="strip"),
        # models whose widths are multiples of 8 only, weights row-major, mixed small batches
        _fwd("packing_ragged", 48, "1000-3080-776-1016", "1..32", mix=5),
        # the same 64 models at moderate batches, between the bandwidth and the compute bound
        _fwd("packing_b33_128", 64, _MLP, "33..128", layout="strip", mix=2),
        # offline batches, compute bound: ragged row counts ...
        _fwd("batch_32_ragged", 32, _MLP, "300..1000", mix=4),
        # ... and the largest, in strips
        _fwd("batch_16_b4096", 16, _MLP, "4096", layout="strip"),
        # the tuning benchmark's step: 8 jobs at batch 64, forward, backward, update
        _train("train_8_b64", 8, _TUNE, 64),
        # the same architecture at a large batch
        _train("train_4_b500", 4, _TUNE, 500),
        # a departure leaves a hole below 4 GB of other jobs' state
        dict(name="compact_4gb", kind="compact", jobs=12, mean_mb=340, mix=1),
        # preemption: 256 MB of state to the host and back
        dict(name="switch_256mb", kind="switch", mb=256),
    ]


def _logint(rng, lo, hi, mult=1):
    v = lo * (hi / lo) ** rng.random()
    return max(lo, min(hi, int(round(v / mult)) * mult))


def draw(rng):
    """Sizes over the ranges of the listed cases; never more work than the largest of its kind."""
    kind = rng.choice(["float", "small", "small", "mid", "large", "train", "train", "compact", "switch"])
    mix = rng.randrange(1 << 20)
    if kind == "float":
        dims = [_logint(rng, 128, 1536, 4) for _ in range(rng.randint(2, 4))]
        top = _logint(rng, 1, 128)
        return _fwd(None, rng.randint(1, 12), "-".join(map(str, dims)), "%d..%d" % (max(1, top // 8), top), dtype="f32",
                    act=rng.choice(["none", "relu", "gelu"]), mix=mix)
    if kind in ("small", "mid", "large"):
        strip = rng.random() < 0.5
        q = 128 if strip else 8
        dims = [_logint(rng, 512, 4096, q) for _ in range(rng.randint(2, 4))]
        size = sum(k * n for k, n in zip(dims, dims[1:]))
        act = rng.choice(["none", "relu", "gelu", "gelu"])
        layout = "strip" if strip else "rows"
        if kind == "small":
            jobs, lo, hi = _logint(rng, 1, 64), 1, _logint(rng, 1, 32)
        elif kind == "mid":
            jobs, lo, hi = _logint(rng, 4, 64), 33, _logint(rng, 40, 128)
        else:
            jobs, lo = _logint(rng, 2, 32), _logint(rng, 129, 2048)
            hi = 2 * lo
        # no more than the packing round's weights and the largest batch's multiply-adds
        jobs = max(1, min(jobs, int(0.6e9 // size), int(0.6e12 // (size * hi))))
        static = kind == "small" and jobs * hi * max(dims) * 4 < (24 << 20) and rng.random() < 0.3
        return _fwd(None, jobs, "-".join(map(str, dims)), "%d..%d" % (lo, hi), act=act, layout=layout, mix=mix, static=static)
    if kind == "train":
        dims = [_logint(rng, 512, 2048, 8) for _ in range(rng.randint(2, 4))] + [_logint(rng, 104, 1000, 8)]
        size = sum(k * n for k, n in zip(dims, dims[1:]))
        rows = _logint(rng, 8, 512)
        jobs = max(1, min(rng.randint(1, 8), int(0.25e11 // (size * rows))))
        return _train(None, jobs, "-".join(map(str, dims)), rows)
    if kind == "compact":
        jobs = rng.randint(4, 16)
        return dict(kind="compact", jobs=jobs, mean_mb=_logint(rng, 8, 3600 // jobs), mix=mix)
    return dict(kind="switch", mb=_logint(rng, 2, 250))


# ---------------------------------------------------------------------------------------------
def _dims(case):
    return [int(v) for v in case["dims"].split("-")]


def _rows(case):
    """Rows of every job in the round (0: the job has no request and is not scheduled)."""
    spec, r = str(case["rows"]), np.random.RandomState(case.get("mix", 1))
    if spec == "poisson":
        rates = np.exp(r.standard_normal(case["jobs"]))
        return [int(min(32, v)) for v in r.poisson(rates * 4.0)]
    if ".." in spec:
        lo, hi = (int(v) for v in spec.split(".."))
        return [int(round(lo * (hi / lo) ** u)) for u in r.random_sample(case["jobs"])]
    return [int(spec)] * case["jobs"]


def _up(v):
    return (v + 255) // 256 * 256


def _gen(seed):
    g = torch.Generator(device="cuda")
    g.manual_seed(seed)
    return g


def _forward_data(case, seed):
    """Per job: the weights (K x N) and the input rows, as the user has them."""
    dims, rows, g = _dims(case), _rows(case), _gen(seed)
    dt = torch.float32 if case["dtype"] == "f32" else torch.bfloat16
    for m in rows:
        W = [(torch.randn(k, n, generator=g, device="cuda") * (k ** -0.5 if case["dtype"] == "f32" else 0.02)).to(dt)
             for k, n in zip(dims, dims[1:])]
        x = torch.randn(max(m, 1), dims[0], generator=g, device="cuda")
        yield m, W, (x if case["dtype"] != "f32" else x.uniform_(-1, 1, generator=g)).to(dt)


def _train_data(case, seed):
    dims, M, g = _dims(case), case["rows"], _gen(seed)
    for _ in range(case["jobs"]):
        W = [torch.randn(k, n, generator=g, device="cuda") * k ** -0.5 for k, n in zip(dims, dims[1:])]
        x = torch.randn(M, dims[0], generator=g, device="cuda").to(torch.bfloat16)
        labels = torch.randint(0, dims[-1], (M,), generator=g, device="cuda", dtype=torch.int32)
        lr = float(10.0 ** (-4.0 + 3.0 * torch.rand(1, generator=g, device="cuda").item()))
        yield W, x, labels, float(np.float32(lr))


def _sizes_mb(case):
    r = np.random.RandomState(case["mix"])
    v = np.exp(0.8 * r.standard_normal(case["jobs"]))
    return [int(round(max(1.0, x))) for x in v / v.mean() * case["mean_mb"]]


class _State:
    """A pool over a buffer of its own, closed with the state."""

    def __init__(self, capacity, policy):
        self.buf = torch.empty(capacity, dtype=torch.uint8, device="cuda")
        self.stream = torch.cuda.current_stream().cuda_stream
        self.pool = salus.Pool(self.buf.data_ptr(), capacity, policy=policy, stream=self.stream)

    def put(self, off, t):
        n = t.numel() * t.element_size()
        self.buf[off:off + n].copy_(t.contiguous().view(torch.uint8).reshape(-1))

    def view(self, off, nbytes, dtype, *shape):
        return self.buf[off:off + nbytes].view(dtype).view(*shape)

    def admit(self, P, E):
        st, j = self.pool.lane_alloc(P, E, 0, 0)
        assert st == salus.OK, self.pool.last_error()
        return j

    def round_of(self, jobs, lanes):
        """What set_pending_many and schedule_into need for a round of these jobs in a pool of that many lanes."""
        n = len(jobs)
        self.ids, self.ones = (ctypes.c_int32 * n)(*jobs), (ctypes.c_uint64 * n)(*[1] * n)
        self.slots, self.lanes, self.n = (salus.Slot * lanes)(), lanes, n

    def schedule(self):
        self.pool.set_pending_many(self.ids, self.ones, self.n)
        assert self.pool.schedule_into(self.slots, self.lanes) == self.n

    def __del__(self):
        torch.cuda.synchronize()
        self.pool.close()


_ACT = {"none": salus.ACT_NONE, "relu": salus.ACT_RELU, "gelu": salus.ACT_GELU}


def _prepare_forward(case, seed):
    dims, rows = _dims(case), _rows(case)
    f32 = case["dtype"] == "f32"
    esz, dt = (4, salus.F32) if f32 else (2, salus.BF16)
    strip = case["layout"] == "strip"
    acts = [_ACT[case["act"]]] * (len(dims) - 2) + [salus.ACT_NONE]
    layers, off = [], 0
    for k, n, a in zip(dims, dims[1:], acts):
        layers.append((k, n, off, a, salus.LAYOUT_STRIP128 if strip else salus.LAYOUT_ROWMAJOR))
        off += _up(k * n * esz)
    P, top = off, max(max(rows), 1)
    y_off = _up(top * dims[0] * esz)
    h_off = y_off + _up(top * dims[-1] * 4)
    E = _up(h_off + max(salus.forward_work_bytes(m, [l[:4] for l in layers], dt) for m in rows + [1]))
    s = _State(case["jobs"] * (P + E), salus.POLICY_PACK)
    items, s.out = [], []
    for m, W, x in _forward_data(case, seed):
        j = s.admit(P, E)
        q = s.pool.job_query(j)
        for (k, n, o, _, _), w in zip(layers, W):
            s.put(q.persist_off + o, w.view(k, n // 128, 128).permute(1, 0, 2) if strip else w)
        s.put(q.lane_off, x)
        if m:
            items.append(dict(job=j, M=m, dtype=dt, layers=layers, x_off=0, y_off=y_off, h_off=h_off))
            s.out.append(s.view(q.lane_off + y_off, m * dims[-1] * 4, torch.float32, m, dims[-1]))
    s.descs, s.keep = salus.Pool.make_descs(items)
    s.round_of([it["job"] for it in items], case["jobs"])
    s.launch = s.pool.grouped_forward_static if case["static"] else s.pool.grouped_forward
    return s


def _prepare_train(case, seed):
    dims, M = _dims(case), case["rows"]
    shapes = list(zip(dims, dims[1:]))
    total = sum(k * n for k, n in shapes)
    layers, wm, wb = [], 0, _up(total * 4)
    for k, n in shapes:                      # all master weights, then all working copies
        layers.append((k, n, wb, wm))
        wm += k * n * 4
        wb += k * n * 2
    P = _up(wb)
    x_off, at = 0, _up(M * dims[0] * 2)
    labels_off, at = at, at + _up(M * 4)
    logits_off, at = at, at + _up(M * dims[-1] * 4)
    loss_off, at = at, at + 256
    E = _up(at + salus.train_work_bytes(M, layers))
    s = _State(case["jobs"] * (P + E), salus.POLICY_PACK)
    items, s.out = [], []
    for W, x, labels, lr in _train_data(case, seed):
        j = s.admit(P, E)
        q = s.pool.job_query(j)
        for (k, n, b, m), w in zip(layers, W):
            s.put(q.persist_off + m, w)
            s.put(q.persist_off + b, w.to(torch.bfloat16))
        s.put(q.lane_off + x_off, x)
        s.put(q.lane_off + labels_off, labels)
        items.append(dict(job=j, M=M, lr=lr, layers=layers, x_off=x_off, labels_off=labels_off, logits_off=logits_off,
                          loss_off=loss_off, work_off=at))
        s.out.append([s.view(q.lane_off + logits_off, M * dims[-1] * 4, torch.float32, M, dims[-1]),
                      s.view(q.lane_off + loss_off, 4, torch.float32, 1),
                      s.view(q.persist_off, total * 4, torch.float32, total),
                      s.view(q.persist_off + _up(total * 4), total * 2, torch.bfloat16, total)])
    s.descs, s.keep = salus.Pool.make_train_descs(items)
    s.round_of([it["job"] for it in items], case["jobs"])
    return s


def _prepare_compact(case, seed):
    mib = 1 << 20
    sizes = [v * mib for v in _sizes_mb(case)]
    E = mib
    s = _State(sum(sizes) + len(sizes) * E, salus.POLICY_PACK)
    s.E, s.order, s.first = E, [], []
    for P in sizes:
        j = s.admit(P, E)
        q = s.pool.job_query(j)
        s.view(q.persist_off, P, torch.int64, P // 8).random_(generator=_gen(seed * 1000 + j))
        s.order.append((j, P))
    s.own = len(sizes)          # jobs 0 .. own - 1 hold data of ours, later ones what the pool held
    return s


def _prepare_switch(case, seed):
    P = case["mb"] << 20
    s = _State(P + (1 << 20), salus.POLICY_PACK)
    s.job = s.admit(P, 1 << 20)
    q = s.pool.job_query(s.job)
    s.view(q.persist_off, P, torch.int64, P // 8).random_(generator=_gen(seed))
    s.P = P
    # the first eviction allocates the pinned buffer that the pool keeps
    assert s.pool.switch_out(s.job) == salus.OK and s.pool.switch_in(s.job) == salus.OK, s.pool.last_error()
    return s


def prepare(case, seed):
    s = {"forward": _prepare_forward, "train": _prepare_train, "compact": _prepare_compact,
         "switch": _prepare_switch}[case["kind"]](case, seed)
    s.kind = case["kind"]
    return s


def run(s):
    if s.kind == "forward":
        s.schedule()
        assert s.launch(s.descs, s.n, s.stream) == salus.OK, s.pool.last_error()
        return s.out
    if s.kind == "train":
        s.schedule()
        assert s.pool.grouped_train_step(s.descs, s.n, s.stream) == salus.OK, s.pool.last_error()
        return s.out
    if s.kind == "compact":
        # the oldest job, which sits lowest, leaves; its hole is closed; a job of its size arrives
        j, P = s.order.pop(0)
        assert s.pool.lane_free(j) >= 0, s.pool.last_error()
        s.pool.compact()
        s.order.append((s.admit(P, s.E), P))
        kept = [(j, P) for j, P in s.order if j < s.own] or s.order[:1]
        return [s.view(s.pool.job_query(j).persist_off, P, torch.int64, P // 8) for j, P in kept]
    assert s.pool.switch_out(s.job) == salus.OK, s.pool.last_error()
    assert s.pool.switch_in(s.job) == salus.OK, s.pool.last_error()
    return s.view(s.pool.job_query(s.job).persist_off, s.P, torch.int64, s.P // 8)


def work(case):
    if case["kind"] == "forward":
        dims, rows = _dims(case), [m for m in _rows(case) if m]
        esz = 4 if case["dtype"] == "f32" else 2
        size = sum(k * n for k, n in zip(dims, dims[1:]))
        return {"bytes": len(rows) * size * esz + sum(rows) * (dims[0] * esz + dims[-1] * 4), "flops": 2 * size * sum(rows)}
    if case["kind"] == "train":
        dims, M = _dims(case), case["rows"]
        size = sum(k * n for k, n in zip(dims, dims[1:]))
        # working weights read and written, master weights read and written; the first layer has no input gradient
        return {"bytes": case["jobs"] * (size * (2 + 2 + 4 + 4) + M * (dims[0] * 2 + 4 + dims[-1] * 4)),
                "flops": case["jobs"] * 2 * M * (3 * size - dims[0] * dims[1])}
    if case["kind"] == "compact":
        return {"bytes": 2 * (sum(_sizes_mb(case)[1:]) << 20), "flops": 0}
    return {"bytes": 2 * (case["mb"] << 20), "flops": 0}


def tolerance(case):
    if case["kind"] in ("compact", "switch"):
        return "exact"
    if case["kind"] == "forward" and case["dtype"] == "f32":
        return {"rel": 4e-6}             # sums of up to 1536 products in 32 bits
    return {"rel": 1e-2, "max": 0.1}     # hidden activations and gradients rounded to bf16


# ---------------------------------------------------------------------------------------------
def _act(z, name):
    if name == "relu":
        return z.clamp_min(0)
    return 0.5 * z * torch.special.erfc(-z * 0.5 ** 0.5) if name == "gelu" else z


def exact(case, seed):
    if case["kind"] == "forward":
        out = []
        for m, W, x in _forward_data(case, seed):
            if not m:
                continue
            h = x.double()
            for l, w in enumerate(W):
                h = h @ w.double()
                if l + 1 < len(W):
                    h = _act(h, case["act"])
            out.append(h)
        return out
    if case["kind"] == "train":
        out = []
        for Wm, x, labels, lr in _train_data(case, seed):
            W = [w.to(torch.bfloat16).double() for w in Wm]
            H = [x.double()]
            for w in W[:-1]:
                H.append((H[-1] @ w).clamp_min(0))
            logits = H[-1] @ W[-1]
            logp = torch.log_softmax(logits, 1)
            at = torch.arange(len(labels), device="cuda")
            d = logp.exp()
            d[at, labels.long()] -= 1
            d /= len(labels)
            new = []
            for l in range(len(W) - 1, -1, -1):
                new.insert(0, (Wm[l].double() - lr * (H[l].t() @ d)).reshape(-1))
                d = (d @ W[l].t()) * (H[l] > 0)
            # the loss is one number: how far it is off is chance, so it is compared by tolerance only
            out.append([logits, None, torch.cat(new), torch.cat(new)])
        return out
    if case["kind"] == "compact":
        sizes = [v << 20 for v in _sizes_mb(case)]
        return [torch.empty(P // 8, dtype=torch.int64, device="cuda").random_(generator=_gen(seed * 1000 + j))
                for j, P in list(enumerate(sizes))[1:]]
    P = case["mb"] << 20
    return torch.empty(P // 8, dtype=torch.int64, device="cuda").random_(generator=_gen(seed))
