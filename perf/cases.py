"""Performance cases: the work a user of the library has it do.

A case is one of five kinds of work, each through the public binding
(paper_2609_09240_amd.tq):

* ``linear``    one packed linear applied to B activation rows, called
                directly: tq_gemv for B = 1, tq_gemm_smallbatch above;
* ``step``      the linear projections of whole decoder layers for B rows, as
                a serving loop runs them: captured once in a HIP graph and
                replayed (``path`` "graph"), or planned once as a chained
                launch (``path`` "chain", B = 1 only);
* ``dequant``   one decoder layer's projections expanded to dense fp16;
* ``codec``     one plane of trits packed, another plane's codes unpacked
                and validated (saving and loading a checkpoint);
* ``quantize``  a dense fp16 weight matrix converted to a packed linear.

Values follow the synthetic workloads of the package: trits with P(0) = 0.4,
scales U(0.01, 0.05), offsets U(-0.01, 0.01), a random two-plane subset,
activations N(0, 1) with 1 % outlier channels on the MLP inputs.  ``f2`` is
the share of groups with a second plane, ``off`` gives every group an
offset, ``f32`` asks for fp32 outputs, ``host`` keeps a host copy of the row
pointers beside the matrix (the binding's default).
"""

import math

import torch

from paper_2609_09240_amd import tq

GROUP = 128
HIDDEN, INTER, KV = 4096, 12288, 1024   # the decoder layer of the package's synthetic workloads


def listed():
    return [
        # The smallest call: a one-plane key/value-sized projection on one
        # activation row.  Launch and latency count, not bytes.
        linear("gemv 1024x4096", 1024, 4096, 1, 0.0, f32=True),
        # Single-user decoding: the linears of 12 layers at batch 1, 10 %
        # two-plane groups, weights larger than the last-level cache.
        step("decode step b1", 12, 1, 0.10),
        # The same work as one chained launch, for programs that cannot replay
        # a graph; the representation with an offset on every group.
        step("decode chain b1 offsets", 4, 1, 0.036, off=True, path="chain"),
        # Few users or speculative drafts: 4 rows.
        step("decode step b4", 4, 4, 0.10),
        # Batched serving, one matrix-core column tile.
        step("decode step b16", 4, 16, 0.10),
        # The largest batch the library takes (also short prompts), with an
        # offset on every group.
        step("decode step b64 offsets", 4, 64, 0.036, off=True),
        # A matrix of no power-of-two size, an odd batch, fp32 outputs, no
        # host row pointers: a caller that only holds device buffers.
        linear("batch33 3000x2560", 3000, 2560, 33, 0.10, off=True, f32=True, host=False),
        # A down projection of a wide MLP: a long row of inputs.
        linear("batch16 4096x20480", 4096, 20480, 16, 0.10),
        # Loading a layer for dense prefill.
        dict(name="dequant layer", kind="dequant", hidden=HIDDEN, inter=INTER, kv=KV, f2=0.10, off=False),
        # Saving and loading the codes of a gate-sized plane.
        dict(name="codec 12288x4096", kind="codec", groups=12288 * 32),
        # Converting a model: a gate-sized matrix, and a small one in the
        # representation with offsets, where launches count.
        dict(name="quantize 12288x4096", kind="quantize", n=12288, k=4096, f2=0.10, iters=4, off=False),
        dict(name="quantize 1024x4096 offsets", kind="quantize", n=1024, k=4096, f2=0.036, iters=4, off=True),
    ]


def linear(name, n, k, b, f2, off=False, f32=False, host=True):
    return dict(name=name, kind="linear", n=n, k=k, b=b, f2=f2, off=off, f32=f32, host=host)


def step(name, layers, b, f2, off=False, path="graph", hidden=HIDDEN, inter=INTER, kv=KV):
    return dict(name=name, kind="step", layers=layers, hidden=hidden, inter=inter, kv=kv, b=b, f2=f2, off=off,
                path=path)


def draw(rng):
    """One more case of the same ranges: any of the kinds, sizes spread over
    their logarithm, odd ones among them."""
    def log_int(lo, hi):
        return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))

    def inputs(lo, hi):
        return GROUP * log_int(lo // GROUP, hi // GROUP)

    f2 = rng.choice([0.0, 0.036, 0.10, 0.10, 0.25])
    off = rng.random() < 0.3
    kind = rng.choice(["linear", "linear", "linear", "step", "step", "dequant", "codec", "quantize"])
    if kind == "linear":
        k = inputs(256, 32768)
        n = log_int(64, min(16384, 4096 * 20480 // k))
        b = rng.choice([1, 2, 3, 4, log_int(2, 64), log_int(5, 64), log_int(5, 64), log_int(17, 64)])
        c = linear("", n, k, b, f2, off=off, f32=rng.random() < 0.4, host=rng.random() < 0.8)
    elif kind == "step":
        hidden = inputs(1024, 4096)
        c = step("", rng.randint(1, 4), rng.choice([1, 1, 2, 4, log_int(5, 64), log_int(5, 64)]), f2, off=off,
                 hidden=hidden, inter=GROUP * max(1, round(hidden * rng.uniform(2.0, 3.0) / GROUP)),
                 kv=GROUP * max(1, hidden // (4 * GROUP)))
        if c["b"] == 1 and rng.random() < 0.4:
            c["path"] = "chain"
    elif kind == "dequant":
        hidden = inputs(512, 4096)
        c = dict(kind=kind, hidden=hidden, inter=GROUP * max(1, round(hidden * rng.uniform(2.0, 3.0) / GROUP)),
                 kv=GROUP * max(1, hidden // (4 * GROUP)), f2=f2, off=off)
    elif kind == "codec":
        c = dict(kind=kind, groups=log_int(1000, 800000))
    else:
        k = inputs(512, 16384)
        c = dict(kind=kind, n=log_int(256, min(16384, 12288 * 4096 // k)), k=k, f2=f2 or 0.10,
                 iters=rng.choice([2, 4, 4, 8]), off=off)
    c.pop("name", None)
    return c


# --------------------------------------------------------------------------
# Inputs, from the seed alone.
# --------------------------------------------------------------------------

def _gen(*key):
    h = 0
    for k in key:
        h = (h * 1000003 + int(k) + 12345) % (1 << 62)
    g = torch.Generator(device="cuda")
    g.manual_seed(h)
    return g


def _trits(shape, g):
    r = torch.randint(0, 10, shape, generator=g, device="cuda", dtype=torch.int8)
    return (r > 6).to(torch.int8) - (r < 3).to(torch.int8)


def _uniform(shape, lo, hi, g):
    return torch.rand(shape, generator=g, device="cuda").mul_(hi - lo).add_(lo).to(torch.float16)


def _rows(k, b, outliers, g):
    x = torch.randn((b, k), generator=g, device="cuda")
    if outliers:
        x[:, torch.randperm(k, generator=g, device="cuda")[:max(1, k // 100)]] *= 20.0
    return x.to(torch.float16)


def _linear_inputs(n, k, f2, off, *key):
    """Unpacked inputs of one packed linear."""
    g = _gen(*key)
    ng = k // GROUP
    nnz = int(f2 * n * ng)
    d = dict(n=n, k=k, nnz=nnz, t0=_trits((n * ng, GROUP), g), s0=_uniform((n, ng), 0.01, 0.05, g))
    if nnz:
        flat = torch.randperm(n * ng, generator=g, device="cuda")[:nnz].sort().values
        d["flat"] = flat
        rowptr = torch.zeros(n + 1, dtype=torch.int64, device="cuda")
        rowptr[1:] = torch.bincount(flat // ng, minlength=n).cumsum(0)
        d["rowptr"] = rowptr.to(torch.int32)
        d["gidx"] = (flat % ng).to(torch.int16)
        d["t1"] = _trits((nnz, GROUP), g)
        d["mu"] = _uniform((nnz,), -0.01, 0.01, g)
        d["s1"] = _uniform((nnz,), 0.01, 0.05, g)
    if off:
        d["mu0"] = _uniform((n, ng), -0.01, 0.01, g)
    return d


def _packed(d, host=True):
    kw = {}
    if d["nnz"]:
        kw = dict(rowptr1=d["rowptr"], gidx1=d["gidx"], codes1=tq.tq_pack(d["t1"]), offset1=d["mu"], scale1=d["s1"])
        if host:
            kw["rowptr1_host"] = d["rowptr"].cpu()
    return tq.PackedLinear(d["n"], d["k"], tq.tq_pack(d["t0"]), d["s0"], offset0=d.get("mu0"), **kw)


def _dense64(d):
    """The weights in 64 bits, by the definition of the representation."""
    w = d["t0"].double() * d["s0"].double().reshape(-1, 1)
    if "mu0" in d:
        w += d["mu0"].double().reshape(-1, 1)
    if d["nnz"]:
        w[d["flat"]] += d["mu"].double().reshape(-1, 1) + d["t1"].double() * d["s1"].double().reshape(-1, 1)
    return w.reshape(d["n"], d["k"])


def _projections(c):
    """(name, outputs, inputs, stage) of one decoder layer; projections of a
    stage read the same activations."""
    h, m, kv = c["hidden"], c["inter"], c["kv"]
    return [("q", h, h, 0), ("k", kv, h, 0), ("v", kv, h, 0), ("o", h, h, 1), ("gate", m, h, 2), ("up", m, h, 2),
            ("down", h, m, 3)]


def _layer_inputs(c, seed, layer):
    return [_linear_inputs(n, k, c["f2"], c["off"], seed, layer, i) for i, (_, n, k, _) in enumerate(_projections(c))]


def _layer_rows(c, seed, layer):
    """Activations of the four stages of a layer."""
    return [_rows(k, c["b"], s >= 2, _gen(seed, layer, 100 + s))
            for s, k in enumerate((c["hidden"], c["hidden"], c["hidden"], c["inter"]))]


def _weights(c, seed):
    g = _gen(seed, 7)
    return torch.randn((c["n"], c["k"]), generator=g, device="cuda").mul_(0.02).to(torch.float16)


# --------------------------------------------------------------------------
# What a program holds before the call, and the call.
# --------------------------------------------------------------------------

def prepare(case, seed):
    c = case
    if c["kind"] == "linear":
        d = _linear_inputs(c["n"], c["k"], c["f2"], c["off"], seed, 0, 0)
        x = _rows(c["k"], c["b"], True, _gen(seed, 0, 100))
        return dict(c, m=_packed(d, c["host"]), x=x[0] if c["b"] == 1 else x)
    if c["kind"] == "step":
        return _prepare_step(c, seed)
    if c["kind"] == "dequant":
        ms = [_packed(d) for d in _layer_inputs(c, seed, 0)]
        return dict(c, ms=ms, ws=[torch.empty((m.n_out, m.n_in), dtype=torch.float16, device="cuda") for m in ms])
    if c["kind"] == "codec":
        n = c["groups"]
        return dict(c, trits=_trits((n, GROUP), _gen(seed, 1)), stored=tq.tq_pack(_trits((n, GROUP), _gen(seed, 2))),
                    codes=torch.empty(26 * n, dtype=torch.uint8, device="cuda"),
                    loaded=torch.empty((n, GROUP), dtype=torch.int8, device="cuda"),
                    bad=torch.zeros(1, dtype=torch.int32, device="cuda"))
    return dict(c, w=_weights(c, seed))


def _prepare_step(c, seed):
    b, projs = c["b"], _projections(c)
    layers, outs = [], []
    for layer in range(c["layers"]):
        ms = [_packed(d) for d in _layer_inputs(c, seed, layer)]
        out = torch.empty(b * sum(m.n_out for m in ms), dtype=torch.float16, device="cuda")
        ys = [y.reshape(b, -1) for y in out.split([b * m.n_out for m in ms])]
        layers.append((ms, _layer_rows(c, seed, layer), ys))
        outs.append(out)
    stages = [[i for i, p in enumerate(projs) if p[3] == s] for s in range(4)]
    if c["path"] == "chain":
        chain = tq.Chain([([ms[i] for i in st], xs[s][0], [ys[i][0] for i in st])
                          for ms, xs, ys in layers for s, st in enumerate(stages)])
        return dict(c, layers=layers, outs=outs, chain=chain)

    def one_step():
        for ms, xs, ys in layers:
            for s, st in enumerate(stages):
                if b == 1:
                    tq.tq_gemv_grouped([ms[i] for i in st], xs[s][0], [ys[i][0] for i in st])
                else:
                    for i in st:
                        tq.tq_gemm_smallbatch(ms[i], xs[s], ys[i])

    side = torch.cuda.Stream()
    side.wait_stream(torch.cuda.current_stream())
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.stream(side):
        one_step()
        side.synchronize()
        graph.capture_begin()
        one_step()
        graph.capture_end()
    torch.cuda.current_stream().wait_stream(side)
    return dict(c, layers=layers, outs=outs, graph=graph)


def run(state):
    s = state
    if s["kind"] == "linear":
        if s["b"] == 1:
            return tq.tq_gemv(s["m"], s["x"], out_f32=s["f32"])
        return tq.tq_gemm_smallbatch(s["m"], s["x"], out_f32=s["f32"])
    if s["kind"] == "step":
        if s["path"] == "chain":
            s["chain"].run()
        else:
            s["graph"].replay()
        return s["outs"]
    if s["kind"] == "dequant":
        return [tq.tq_unpack_fp16(m, w) for m, w in zip(s["ms"], s["ws"])]
    if s["kind"] == "codec":
        return dict(codes=tq.tq_pack(s["trits"], s["codes"], s["bad"]),
                    trits=tq.tq_unpack(s["stored"], s["groups"], s["loaded"], s["bad"]),
                    bad=tq.tq_validate(s["stored"], s["groups"], s["bad"]))
    p = tq.quantize_linear(s["w"], f2=s["f2"], iters=s["iters"], group_offsets=s["off"])
    out = dict(codes0=p.codes0, scale0=p.scale0, rowptr1=p.rowptr1, rowptr1_host=p.rowptr1_host, gidx1=p.gidx1,
               codes1=p.codes1, offset1=p.offset1, scale1=p.scale1)
    if s["off"]:
        out["offset0"] = p.offset0
    return out


# --------------------------------------------------------------------------
# Work, tolerance and the same values in 64 bits.
# --------------------------------------------------------------------------

def _packed_bytes(n, k, f2, off):
    ng = n * (k // GROUP)
    nnz = int(f2 * ng)
    return (28 + (2 if off else 0)) * ng + (4 * (n + 1) + 32 * nnz if nnz else 0)


def work(case):
    """Each input read once, each output written once; two flops per weight
    and activation row."""
    c = case
    if c["kind"] == "linear":
        return dict(bytes=_packed_bytes(c["n"], c["k"], c["f2"], c["off"]) + 2 * c["b"] * c["k"]
                    + (4 if c["f32"] else 2) * c["b"] * c["n"], flops=2 * c["b"] * c["n"] * c["k"])
    if c["kind"] == "step":
        ps = _projections(c)
        by = sum(_packed_bytes(n, k, c["f2"], c["off"]) + 2 * c["b"] * n for _, n, k, _ in ps)
        by += 2 * c["b"] * (3 * c["hidden"] + c["inter"])
        return dict(bytes=c["layers"] * by, flops=c["layers"] * 2 * c["b"] * sum(n * k for _, n, k, _ in ps))
    if c["kind"] == "dequant":
        ps = _projections(c)
        return dict(bytes=sum(_packed_bytes(n, k, c["f2"], c["off"]) + 2 * n * k for _, n, k, _ in ps), flops=0)
    if c["kind"] == "codec":
        return dict(bytes=c["groups"] * (154 + 154 + 26), flops=0)
    nk = c["n"] * c["k"]
    return dict(bytes=2 * nk + _packed_bytes(c["n"], c["k"], c["f2"], c["off"]), flops=8 * nk)


def tolerance(case):
    c = case
    # About four times the distance from the 64-bit values.  fp32 outputs at
    # batch 1 show fp32 sums only (7e-8); a batch may round the weights of
    # two-plane and offset groups to fp16 (2.3e-4), and fp16 outputs are one
    # rounding (2.1e-4 to 3e-4).
    if c["kind"] == "linear" and c["b"] == 1 and c["f32"]:
        return {"rel": 8e-7}
    if c["kind"] in ("linear", "step"):
        return {"rel": 1.2e-3}
    return "exact"   # codes, trits and single roundings of uniquely defined values


def exact(case, seed):
    c = case
    if c["kind"] == "linear":
        w = _dense64(_linear_inputs(c["n"], c["k"], c["f2"], c["off"], seed, 0, 0))
        y = _rows(c["k"], c["b"], True, _gen(seed, 0, 100)).double() @ w.t()
        return y[0] if c["b"] == 1 else y
    if c["kind"] == "step":
        outs = []
        for layer in range(c["layers"]):
            xs = _layer_rows(c, seed, layer)
            outs.append(torch.cat([(xs[p[3]].double() @ _dense64(d).t()).reshape(-1)
                                   for p, d in zip(_projections(c), _layer_inputs(c, seed, layer))]))
        return outs
    if c["kind"] == "dequant":
        return [_dense64(d) for d in _layer_inputs(c, seed, 0)]
    if c["kind"] == "codec":
        return None
    return _exact_quantize(c, seed)


def _threshold(v):
    d = 0.75 * v.abs().mean(1, keepdim=True)
    return (v > d).double() - (v < -d).double()


def _scale(t, v):
    n = t.abs().sum(1, keepdim=True)
    return torch.where(n > 0, (t * v).sum(1, keepdim=True) / n.clamp(min=1), torch.zeros_like(n))


def _exact_quantize(c, seed):
    """Scales and offsets in 64 bits (the codes are whole numbers)."""
    w = _weights(c, seed).double().reshape(-1, GROUP)
    mu = w.mean(1, keepdim=True) if c["off"] else torch.zeros((w.shape[0], 1), dtype=torch.float64, device="cuda")
    t = _threshold(w - mu)
    s0 = _scale(t, w - mu)
    for _ in range(c["iters"] if c["off"] else 0):
        mu = (w - s0 * t).mean(1, keepdim=True)
        s0 = _scale(t, w - mu)
    energy = (w - mu - s0 * t).square().sum(1)
    nnz = int(math.floor(c["f2"] * c["n"] * (c["k"] // GROUP)))
    sel = torch.sort(energy, descending=True, stable=True).indices[:nnz].sort().values
    v = w[sel]
    m2 = v.mean(1, keepdim=True)
    a = _threshold(v - m2)
    sa = _scale(a, v - m2)
    b = _threshold(v - m2 - sa * a)
    sb = _scale(b, v - m2 - sa * a)
    for _ in range(c["iters"]):
        m2 = (v - sa * a - sb * b).mean(1, keepdim=True)
        sa = _scale(a, v - m2 - sb * b)
        sb = _scale(b, v - m2 - sa * a)
    s0[sel] = sa
    out = dict(codes0=None, scale0=s0.reshape(c["n"], -1), rowptr1=None, rowptr1_host=None, gidx1=None, codes1=None,
               scale1=sb[:, 0])
    if c["off"]:
        mu[sel] = m2
        out["offset0"] = mu.reshape(c["n"], -1)
        out["offset1"] = torch.zeros_like(m2[:, 0])
    else:
        out["offset1"] = m2[:, 0]
    return out
