"""The work a training job hands to this library, as measurable cases.

Every case goes through the public entry points of `paper_1512_06216_amd.binding` the way a data-parallel
worker's training loop calls them: the per-worker factor blocks (or gradient copies), weights and momentum are
in device memory, the plan, stacked buffers, workspace and marshalled iteration are kept from step to step, and
one pass is one step's synchronisation of one layer or of a whole network.  M = inputs and N = outputs of a
fully-connected layer, B = batch per worker, P = workers, K = P*B stacked samples.
"""
import math

import torch

from paper_1512_06216_amd import binding as psd
from paper_1512_06216_amd import inputs

LR, MU, WD = inputs.LR, inputs.MU, 5e-4      # step, momentum and weight decay of a Caffe-style training run

CNN_CONV = ",".join(str(n) for n in inputs.conv_sizes())
CNN_FC = ",".join("%dx%d" % s for s in inputs.FC_SHAPES)

# what the largest listed cases take: a drawn case stays below these
MAX_FLOPS = {"f32": 2.3e11, "bf16": 4.2e11}
MAX_BYTES = 1.8e9


def listed():
    fc = dict(kind="fc", B=256, P=8, scratch="workspace", errors="gauss")
    return [
        # the smallest call: a little classifier head on four workers, where launches and host work are everything
        dict(fc, name="tiny_fc_f32", M=256, N=128, B=32, P=4, dtype="f32"),
        # a 1000-way classifier on pooled features at batch 32 per worker: few tiles, short contraction
        dict(fc, name="googlenet_fc_bf16", M=1024, N=1000, B=32, dtype="bf16"),
        # AlexNet's last layer with fp32 factors (the paper's own precision)
        dict(fc, name="classifier_fc_f32", M=4096, N=1000, dtype="f32"),
        # AlexNet's largest layer
        dict(fc, name="fc6_bf16", M=9216, N=4096, dtype="bf16"),
        # the 21 841-way ImageNet-22K classifier; its errors are softmax minus one-hot
        dict(fc, name="cls22k_bf16", M=4096, N=21841, dtype="bf16", errors="softmax"),
        # the same on the 3000-wide network: rows of W that start in the middle of a cache line
        dict(fc, name="in22k_cls_bf16", M=3000, N=21841, dtype="bf16", errors="softmax"),
        # VGG-16's first fully-connected layer from blocks the senders rounded, read where they were received
        dict(kind="blocks", name="vgg_fc6_blocks_bf16", M=25088, N=4096, B=256, P=8, dtype="bf16", errors="gauss"),
        # the five convolution layers of AlexNet, ready together, one parameter-server launch
        dict(kind="conv", name="conv_layers", sizes=CNN_CONV, P=8, S=8),
        # a large layer through the parameter server: dense copies of fc6's gradient
        dict(kind="dense", name="dense_fc6", n=9216 * 4096, P=8, S=8),
        # one whole training step of AlexNet, all eight layers, each on its own stream; bf16 and fp32 factors
        dict(kind="iteration", name="cnn_bf16", conv=CNN_CONV, fc=CNN_FC, B=256, P=8, S=8, dtype="bf16"),
        dict(kind="iteration", name="cnn_f32", conv=CNN_CONV, fc=CNN_FC, B=256, P=8, S=8, dtype="f32"),
        # AlexNet's last layer trained under bounded staleness
        dict(kind="ssp", name="ssp_classifier_bf16", M=4096, N=1000, B=256, P=8, dtype="bf16", errors="gauss", staleness=2),
    ]


# ---------------------------------------------------------------------------------------------- drawn cases
def _spread(rng, lo, hi):
    """Spread over the logarithm of [lo, hi]; half of the draws are multiples of 32, the rest whatever comes."""
    n = int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))
    if rng.random() < 0.5 and n >= 64:
        n = n // 32 * 32
    return max(lo, min(hi, n))


def _draw_fc(rng, kind):
    c = dict(kind=kind, M=_spread(rng, 64, 25088), N=_spread(rng, 64, 21841), B=_spread(rng, 16, 256), P=rng.choice([2, 4, 8, 16]),
             dtype=rng.choice(["f32", "bf16", "bf16"]), errors=rng.choice(["gauss", "softmax"]))
    if kind == "fc":
        c["scratch"] = rng.choice(["workspace", "workspace", "static", "none"])
    elif kind == "ssp":
        c["staleness"] = rng.randint(0, 4)
    elif kind == "blocks":
        # what can be read in place: whole k-stages in a block; dense fp32 rows a multiple of 16 bytes
        q = 32 if c["dtype"] == "bf16" else 16
        c["B"] = max(q, c["B"] // q * q)
        if c["dtype"] == "f32":
            c["M"], c["N"] = c["M"] // 4 * 4, c["N"] // 4 * 4
    return c


def _draw_once(rng):
    kind = rng.choice(["fc", "fc", "fc", "blocks", "dense", "conv", "iteration", "ssp"])
    if kind == "dense":
        n = _spread(rng, 500, 60_000_000)
        return dict(kind=kind, n=n, P=rng.choice([1, 2, 3, 4, 6, 8, 8, 12, 16]), S=rng.choice([1, 4, 8, 16, 61]))
    if kind == "conv":
        sizes = [_spread(rng, 500, 2_400_000) for _ in range(rng.randint(2, 8))]
        return dict(kind=kind, sizes=",".join(str(n) for n in sizes), P=rng.choice([2, 4, 5, 8, 16]), S=rng.choice([1, 4, 8]))
    if kind == "iteration":
        sizes = [_spread(rng, 500, 1_500_000) for _ in range(rng.randint(2, 6))]
        w = [_spread(rng, 128, 9216)] + [_spread(rng, 64, 4096) for _ in range(rng.randint(1, 3))]
        return dict(kind=kind, conv=",".join(str(n) for n in sizes), fc=",".join("%dx%d" % (a, b) for a, b in zip(w, w[1:])),
                    B=_spread(rng, 16, 256), P=rng.choice([2, 4, 8]), S=rng.choice([1, 4, 8]), dtype=rng.choice(["f32", "bf16"]))
    return _draw_fc(rng, kind)


def draw(rng):
    while True:
        c = _draw_once(rng)
        w = work(c)
        if w["flops"] <= MAX_FLOPS[c.get("dtype", "f32")] and w["bytes"] <= MAX_BYTES:
            if c["kind"] not in ("fc", "ssp", "blocks") or c["M"] * c["N"] <= 110_000_000:
                return c


# ---------------------------------------------------------------------------------------------- inputs
class _Maker:
    """Seeded synthetic training data on the GPU: activations after a ReLU, errors, weights, gradient copies."""

    def __init__(self, seed):
        self.gen = torch.Generator(device="cuda").manual_seed(int(seed))

    def normal(self, shape, std):
        return torch.randn(shape, generator=self.gen, device="cuda", dtype=torch.float32).mul_(std)

    def activations(self, B, M):
        return self.normal((B, M), 1.0).relu_()

    def errors(self, B, N, how):
        if how == "gauss":
            return self.normal((B, N), 1e-3)
        e = torch.softmax(self.normal((B, N), 1.0), dim=1)
        y = torch.randint(0, N, (B, 1), generator=self.gen, device="cuda")
        return e.scatter_add_(1, y, torch.full((B, 1), -1.0, device="cuda")).div_(B)

    def params(self, shape):
        return self.normal(shape, 1e-2), self.normal(shape, 1e-3)      # weights and momentum in mid-training


def _dtype(case):
    return psd.F32 if case["dtype"] == "f32" else psd.BF16


def _ints(text):
    return [int(x) for x in text.split(",") if x]


def _shapes(text):
    return [tuple(int(v) for v in x.split("x")) for x in text.split(",")]


def _factors(mk, case, M, N):
    how = case.get("errors", "gauss")
    return ([mk.errors(case["B"], N, how) for _ in range(case["P"])], [mk.activations(case["B"], M) for _ in range(case["P"])])


_layer_streams = []        # one stream per layer position, kept for the life of the program


def _streams(n):
    while len(_layer_streams) < n:
        _layer_streams.append(torch.cuda.Stream())
    return _layer_streams[:n]


# ---------------------------------------------------------------------------------------------- one FC layer
def _prepare_fc(case, mk):
    M, N, dt = case["M"], case["N"], _dtype(case)
    plan = psd.plan_layer(psd.LAYER_FC, M, N, case["B"], case["P"])
    delta, act = _factors(mk, case, M, N)
    U, ldu, V, ldv = psd.alloc_factors(plan, dt)
    W, Mom = mk.params((N, M))
    bias, mom_bias = mk.params((N,))
    ws = psd.alloc_workspace(plan, dt) if case["scratch"] == "workspace" else None
    return dict(kind="fc", plan=plan, dt=dt, delta=delta, act=act, U=U, ldu=ldu, V=V, ldv=ldv, W=W, Mom=Mom, bias=bias,
                mom_bias=mom_bias, ws=ws, static=case["scratch"] == "static" and _static_fits(plan, dt))


def _static_fits(plan, dt):
    return psd.sfb_workspace_bytes(plan, dt) <= psd.STATIC_SCRATCH_BYTES


def _run_fc(s):
    psd.pack_factors(s["plan"], s["delta"], s["act"], s["dt"], s["U"], s["ldu"], s["V"], s["ldv"])
    if s["static"]:
        psd.sync_fc_sfb_static(s["plan"], s["dt"], s["U"], s["ldu"], s["V"], s["ldv"], s["W"], s["Mom"], LR, MU, wd=WD)
    else:
        psd.sync_fc_sfb(s["plan"], s["dt"], s["U"], s["ldu"], s["V"], s["ldv"], s["W"], s["Mom"], LR, MU, wd=WD,
                        workspace=s["ws"])
    psd.sync_fc_bias(s["plan"], s["dt"], s["U"], s["ldu"], s["bias"], s["mom_bias"], LR, MU, wd=WD)
    return {k: s[k] for k in ("U", "V", "W", "Mom", "bias", "mom_bias")}


# ---------------------------------------------------------------------------------------------- blocks in place
def _prepare_blocks(case, mk):
    M, N, dt = case["M"], case["N"], _dtype(case)
    plan = psd.plan_layer(psd.LAYER_FC, M, N, case["B"], case["P"])
    delta, act = _factors(mk, case, M, N)
    W, Mom = mk.params((N, M))
    ldu = ldv = 0
    if dt == psd.BF16:                           # every sender rounds its own block before it sends it
        one = psd.plan_layer(psd.LAYER_FC, M, N, case["B"], 1)
        for p in range(case["P"]):
            U, ldu, V, ldv = psd.alloc_factors(one, dt)
            psd.pack_factors(one, [delta[p]], [act[p]], dt, U, ldu, V, ldv)
            delta[p], act[p] = U, V
    return dict(kind="blocks", plan=plan, dt=dt, delta=delta, act=act, ldu=ldu, ldv=ldv, W=W, Mom=Mom)


def _run_blocks(s):
    psd.sync_fc_sfb_blocks(s["plan"], s["dt"], s["delta"], s["ldu"], s["act"], s["ldv"], s["W"], s["Mom"], LR, MU, wd=WD)
    return {"W": s["W"], "Mom": s["Mom"]}


# ---------------------------------------------------------------------------------------------- staleness
def _prepare_ssp(case, mk):
    M, N, dt, stale = case["M"], case["N"], _dtype(case), case["staleness"]
    plan = psd.plan_layer(psd.LAYER_FC, M, N, case["B"], case["P"])
    delta, act = _factors(mk, case, M, N)
    W, Mom = mk.params((N, M))
    s = dict(kind="ssp", plan=plan, delta=delta, act=act, W=W, Mom=Mom, ws=psd.alloc_workspace(plan, dt),
             ssp=psd.SspFc(plan, dt, stale))
    for _ in range(stale):                       # the clocks of a running job: an update falls due in every pass
        _run_ssp(s)
    return s


def _run_ssp(s):
    s["ssp"].clock(s["delta"], s["act"], s["W"], s["Mom"], LR, MU, wd=WD, workspace=s["ws"])
    return {"W": s["W"], "Mom": s["Mom"]}


# ---------------------------------------------------------------------------------------------- parameter server
def _prepare_dense(case, mk):
    n = case["n"]
    G = [mk.normal((n,), 1e-3) for _ in range(case["P"])]
    W, Mom = mk.params((n,))
    return dict(kind="dense", G=G, W=W, Mom=Mom, S=min(case["S"], n))


def _run_dense(s):
    psd.sync_dense_ps(s["G"], s["W"], s["Mom"], LR, MU, s["S"], wd=WD)
    return {"W": s["W"], "Mom": s["Mom"]}


def _prepare_conv(case, mk):
    layers = []
    for n in _ints(case["sizes"]):
        G = [mk.normal((n,), 1e-3) for _ in range(case["P"])]
        layers.append((G, *mk.params((n,)), min(case["S"], n)))
    return dict(kind="conv", layers=layers, multi=psd.DenseMulti(layers))


def _run_conv(s):
    s["multi"].run(LR, MU, wd=WD)
    return {"W": [x[1] for x in s["layers"]], "Mom": [x[2] for x in s["layers"]]}


# ---------------------------------------------------------------------------------------------- a whole step
def _prepare_iteration(case, mk):
    dt, P, B = _dtype(case), case["P"], case["B"]
    convs, fcs = _ints(case["conv"]), _shapes(case["fc"])
    streams = _streams(len(convs) + len(fcs))
    ready = torch.cuda.Event()                   # "the gradients of this step exist"
    ready.record()
    tasks = []
    for n in convs:
        plan = psd.plan_layer(psd.LAYER_CONV, n, 1, B, P)
        W, Mom = mk.params((n,))
        tasks.append(dict(plan=plan, S=min(case["S"], n), G=[mk.normal((n,), 1e-3) for _ in range(P)], W=W, Mom=Mom))
    for M, N in fcs:
        plan = psd.plan_layer(psd.LAYER_FC, M, N, B, P)
        delta, act = _factors(mk, case, M, N)
        U, ldu, V, ldv = psd.alloc_factors(plan, dt)
        W, Mom = mk.params((N, M))
        tasks.append(dict(plan=plan, factor_dtype=dt, delta=delta, act=act, U=U, ldu=ldu, V=V, ldv=ldv, W=W, Mom=Mom,
                          workspace=psd.alloc_workspace(plan, dt)))
    for t, st in zip(tasks, streams):
        t["stream"], t["ev_ready"] = st, ready.cuda_event
    return dict(kind="iteration", tasks=tasks, streams=streams, ready=ready, it=psd.Iteration(tasks))


def _run_iteration(s):
    here = torch.cuda.current_stream()
    s["ready"].record(here)
    s["it"].run(LR, MU, wd=WD)
    for st in s["streams"]:                      # the next forward pass reads every layer's weights
        here.wait_stream(st)
    return {"W": [t["W"] for t in s["tasks"]], "Mom": [t["Mom"] for t in s["tasks"]],
            "U": [t["U"] for t in s["tasks"] if "U" in t], "V": [t["V"] for t in s["tasks"] if "V" in t]}


_PREPARE = dict(fc=_prepare_fc, blocks=_prepare_blocks, ssp=_prepare_ssp, dense=_prepare_dense, conv=_prepare_conv,
                iteration=_prepare_iteration)
_RUN = dict(fc=_run_fc, blocks=_run_blocks, ssp=_run_ssp, dense=_run_dense, conv=_run_conv, iteration=_run_iteration)


def prepare(case, seed):
    return _PREPARE[case["kind"]](case, _Maker(seed))


def run(state):
    return _RUN[state["kind"]](state)


# ---------------------------------------------------------------------------------------------- work and tolerance
def _dense_work(n, P):
    return n * (4 * P + 16), n * (P + 6)


def _fc_work(M, N, K, es, packed):
    """Weights and momentum read and written, the contraction, and the factors: fp32 blocks in, stacked matrices out, or
    (packed = False) blocks of the factor type read once."""
    factors = K * (M + N)
    return 16 * M * N + factors * (4 + es if packed else es), 2 * M * N * K + 6 * M * N


def work(case):
    kind, es = case["kind"], 2 if case.get("dtype") == "bf16" else 4
    if kind == "dense":
        b, f = _dense_work(case["n"], case["P"])
    elif kind == "conv":
        per = [_dense_work(n, case["P"]) for n in _ints(case["sizes"])]
        b, f = sum(x[0] for x in per), sum(x[1] for x in per)
    elif kind == "iteration":
        per = [_dense_work(n, case["P"]) for n in _ints(case["conv"])]
        per += [_fc_work(M, N, case["P"] * case["B"], es, True) for M, N in _shapes(case["fc"])]
        b, f = sum(x[0] for x in per), sum(x[1] for x in per)
    else:
        K = case["P"] * case["B"]
        b, f = _fc_work(case["M"], case["N"], K, es, kind != "blocks")
        if kind == "fc":                         # the bias: its sum reads the stacked errors that are there already
            b, f = b + 16 * case["N"], f + case["N"] * (K + 6)
        elif kind == "ssp" and case["staleness"] > 0:        # the factors of an earlier clock are what is contracted
            b += K * (case["M"] + case["N"]) * es
    return {"bytes": b, "flops": f}


def tolerance(case):
    # sums and products in fp32 over the very same (rounded) inputs: only the order of additions may differ
    return {"rel": 1e-5}
