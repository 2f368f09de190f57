"""What this framework's speed is measured on: passes of requests through collaborating experts, by the public binding.

A pass is what a serving loop does: coe_submit the requests, coe_step until every request has left its last expert,
coe_collect logits and paths.  Before it, a program has built a context, registered its experts' weights and set the
dependency graph.  Request images lie in device memory, except where a case says that they come from the host.

Routing heads are fitted so that an image's class decides its route with a wide margin, as a trained classifier's does:
with random heads the two best logits of many requests differ by less than bf16 rounding, and any two correct
implementations would send some requests to different experts.  The fit uses plain fp32 torch arithmetic on a few
prototype images and nothing of the framework.  The experts whose logits a request ends with keep random heads.
"""
import math

import numpy as np
import torch
import torch.nn.functional as F

import coe_workloads as W
from paper_2503_02354_amd import binding as B

STATIC_INTS = 1 << 20   # what coe_regroup_static's scratch holds: ceil(n / 256) * experts int32
GRID = 4            # a class's prototype has GRID x GRID cells per channel, one N(0,1) value each
NOISE = 0.5         # standard deviation of the pixel noise on top, as in the repository's structured workloads
STAGES = {"tree18": 2, "tree50": 2, "dag": 3, "vit": 2, "detect": 2, "tiny": 2}


def listed():
    return [
        # one request through a classifier and the expert it selects: the latency of an idle service
        dict(name="tree18_1", kind="tree18", n=1, experts=16, hw=224, host=False),
        # a handful of requests over 15 leaf experts: every group has one to four
        dict(name="tree18_29", kind="tree18", n=29, experts=16, hw=224, host=False),
        # an ordinary batch whose images arrive in host memory, as from a camera or a decoder
        dict(name="tree18_host_500", kind="tree18", n=500, experts=16, hw=224, host=True),
        # the benchmark's workload: 4096 requests, 16 ResNet-18-shaped experts, all resident
        dict(name="tree18_4096", kind="tree18", n=4096, experts=16, hw=224, host=False),
        # ResNet-50-shaped experts under a device cache that holds a third of them, arrivals of 256 with a stage after
        # each, an arranging window, prefetch and three executors: expert switching under load
        dict(name="tree50_cap_2048", kind="tree50", n=2048, experts=18, cap=6, arrival=256, hw=224),
        # three stages over two architectures with shared downstream experts and skewed groups
        dict(name="dag_1500", kind="dag", n=1500, tiers="4,10,20", hw=224),
        # transformer-shaped experts, few requests
        dict(name="vit_5", kind="vit", n=5, experts=3, cap=0, hw=224),
        # transformer-shaped experts, more of them than the device cache holds
        dict(name="vit_cap_777", kind="vit", n=777, experts=7, cap=4, hw=224),
        # classifiers that route to shared detector-shaped experts
        dict(name="detect_1000", kind="detect", n=1000, classifiers=2, detectors=4, hw=224),
        # small fp32 experts on 64 x 64 images
        dict(name="tiny_fp32_256", kind="tiny", n=256, experts=4, hw=64),
        # the regroup by itself, on device arrays, for a model of more than 300 experts
        dict(name="regroup_100003", kind="regroup", n=100003, experts=370, live=0.8),
    ]


def _spread(rng, lo, hi):
    """An integer whose logarithm is uniform over the range."""
    return max(lo, min(hi, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


def draw(rng):
    kind = rng.choice(["tree18", "tree18", "tree50", "dag", "vit", "detect", "tiny", "regroup"])
    hw = rng.choice([64, 128, 192, 224, 224, 224])
    if kind == "tree18":
        return dict(kind=kind, n=_spread(rng, 1, 3000), experts=rng.randint(4, 16), hw=hw, host=rng.random() < 0.25)
    if kind == "tree50":
        experts = rng.randint(6, 18)
        arrival = _spread(rng, 32, 512)
        return dict(kind=kind, n=min(1800, arrival * rng.randint(1, 7) + rng.randint(0, 31)), experts=experts,
                    cap=rng.choice([0, 6]), arrival=arrival, hw=hw)
    if kind == "dag":
        return dict(kind=kind, n=_spread(rng, 8, 1400), tiers="%d,%d,%d" % (rng.randint(2, 4), rng.randint(5, 10), rng.randint(8, 20)), hw=hw)
    if kind == "vit":
        experts = rng.randint(3, 7)
        return dict(kind=kind, n=_spread(rng, 1, 700), experts=experts, cap=rng.choice([0, 4]), hw=hw)
    if kind == "detect":
        return dict(kind=kind, n=_spread(rng, 1, 900), classifiers=rng.randint(1, 2), detectors=rng.randint(2, 4), hw=hw)
    if kind == "tiny":
        return dict(kind=kind, n=_spread(rng, 1, 1024), experts=rng.randint(3, 5), hw=rng.choice([32, 48, 64]))
    n = _spread(rng, 1, 131072)
    most = min(2048, STATIC_INTS // ((n + 255) // 256))
    return dict(kind=kind, n=n, experts=_spread(rng, 2, most), live=rng.choice([0.5, 0.8, 1.0]))


# ---- the model a case serves -----------------------------------------------------------------------------------
def _model(case):
    """(architectures, architecture of every expert, successor lists, usage probabilities, probabilities of the first
    experts, probabilities of the image classes).  Class c takes successor c modulo their number."""
    kind, hw = case["kind"], case["hw"]
    if kind in ("tree18", "tree50", "vit", "tiny"):
        e, first = case["experts"], [1.0]
        make = {"tree18": W.resnet18, "tree50": W.resnet50, "vit": W.vit}.get(kind)
        archs, e_arch = [make(e, hw) if make else W.tiny_cnn(max(4, e), hw)], [0] * e
        lists = [list(range(1, e))] + [[] for _ in range(e - 1)]
        fan = e - 1
    elif kind == "dag":
        n1, n2, n3 = (int(v) for v in case["tiers"].split(","))
        fan = 5
        lists = [[n1 + (i * n2 // n1 + d) % n2 for d in range(fan)] for i in range(n1)]
        lists += [[n1 + n2 + (j * n3 // n2 + d) % n3 for d in range(fan)] for j in range(n2)]
        lists += [[] for _ in range(n3)]
        archs, e_arch = [W.resnet18(fan + 1, hw), W.resnet50(fan + 1, hw)], [e % 2 for e in range(n1 + n2 + n3)]
        first = list(W.zipf_probs(n1, 1.2))
    else:
        n1, n3 = case["classifiers"], case["detectors"]
        fan = min(6, n3)
        lists = [[n1 + (i * n3 // n1 + d) % n3 for d in range(fan)] for i in range(n1)] + [[] for _ in range(n3)]
        archs, e_arch = [W.resnet18(fan + 2, hw), W.detector(27, hw)], [0] * n1 + [1] * n3
        first = list(W.zipf_probs(n1, 1.2))
    classes = list(W.zipf_probs(fan, 1.1)) if kind in ("tree50", "dag") else [1.0 / fan] * fan
    prob = [0.0] * len(lists)
    for e0, pe in enumerate(first):
        for c, pc in enumerate(classes):
            e = e0
            while True:
                prob[e] += pe * pc
                if not lists[e]:
                    break
                e = lists[e][c % len(lists[e])]
    return archs, e_arch, lists, prob, first, classes


def _images(proto, cls, hw, gen):
    up = proto.repeat_interleave(hw // GRID, 1).repeat_interleave(hw // GRID, 2)
    out = torch.empty((len(cls), hw, hw, 3), dtype=torch.bfloat16, device="cuda")
    for s in range(0, len(cls), 256):
        x = up[cls[s:s + 256]]
        out[s:s + 256] = x + NOISE * torch.randn(x.shape, generator=gen, device="cuda")
    return out


def _features(arch, blob, x):
    """What the head of `arch` multiplies its weights with, for images x: fp32 throughout."""
    specs, _ = W.blob_layout(arch)
    dt = torch.bfloat16 if arch.dtype == W.DT_BF16 else torch.float32
    t = {(s.layer, s.name): blob[s.offset:s.offset + s.nbytes].view(dt if s.is_param_dtype else torch.float32).float().view(s.shape) for s in specs}
    act = {0: lambda v: v, 1: F.relu, 2: F.gelu, 3: F.silu}
    buf = {0: x.float().permute(0, 3, 1, 2).contiguous()}                      # [n][c][h][w]
    for i, layer in enumerate(arch.layers):
        op, src, dst, res, k, r, s, stride, pad, a, aux, _ = (int(v) for v in layer)
        v = buf[src]
        n, c, h, w = v.shape
        if op == W.OP_CONV:
            cols = v[:, :, ::stride, ::stride].reshape(n, c, -1) if r == 1 else F.unfold(v, (r, s), padding=pad, stride=stride)
            wt = t[i, "w"].permute(0, 3, 1, 2).reshape(k, -1)
            y = torch.matmul(wt, cols.transpose(0, 1).reshape(cols.shape[1], -1)).view(k, n, -1).transpose(0, 1)
            y = (y + t[i, "b"][:, None]).reshape(n, k, (h + 2 * pad - r) // stride + 1, (w + 2 * pad - s) // stride + 1)
            buf[dst] = act[a](y + buf[res] if res >= 0 else y)
        elif op == W.OP_MAXPOOL:
            buf[dst] = F.max_pool2d(v, (r, s), stride, pad)
        elif op == W.OP_TOKENS:
            tok = torch.cat([t[i, "cls"].expand(n, 1, c), v.flatten(2).transpose(1, 2)], 1) + t[i, "pos"]
            buf[dst] = tok.transpose(1, 2)[..., None]
        elif op == W.OP_LAYERNORM:
            y = F.layer_norm(v[..., 0].transpose(1, 2), (c,), t[i, "gamma"], t[i, "beta"], 1e-6)
            buf[dst] = y.transpose(1, 2)[..., None]
        elif op == W.OP_ATTENTION:
            q, key, val = (z.reshape(n, aux, c // 3 // aux, h) for z in v[..., 0].chunk(3, 1))
            p = torch.softmax(torch.matmul(q.transpose(2, 3).contiguous(), key) / math.sqrt(c // 3 // aux), -1)
            buf[dst] = torch.matmul(val, p.transpose(2, 3).contiguous()).reshape(n, c // 3, h, 1)
        elif op == W.OP_HEAD:
            return v.mean((2, 3))
        else:
            return F.layer_norm(v[:, :, 0, 0], (c,), t[i, "gamma"], t[i, "beta"], 1e-6)


def _blob(arch, gen):
    """Random weights in the repository's distributions (coe_workloads.make_expert_blob), drawn on the GPU."""
    specs, nbytes = W.blob_layout(arch)
    blob = torch.zeros(nbytes, dtype=torch.uint8, device="cuda")
    for s in specs:
        op, act, res = int(arch.layers[s.layer][0]), int(arch.layers[s.layer][9]), int(arch.layers[s.layer][3])
        mean, std = {"b": (0.0, W.BIAS_STD), "gamma": (1.0, 0.1), "beta": (0.0, 0.1), "cls": (0.0, 0.5), "pos": (0.0, 0.5)}.get(s.name, (0.0, 0.0))
        if s.name == "w":
            he = op == W.OP_CONV and arch.name != "vit" and (act in (W.ACT_RELU, W.ACT_SILU) or res >= 0)
            std = math.sqrt((2.0 if he else 1.0) / math.prod(s.shape[1:])) * (arch.gains[s.layer] if op == W.OP_CONV else 1.0)
        v = mean + std * torch.randn(math.prod(s.shape), generator=gen, device="cuda")
        v = v.to(torch.bfloat16) if s.is_param_dtype and arch.dtype == W.DT_BF16 else v
        blob[s.offset:s.offset + s.nbytes] = v.view(torch.uint8)
    return blob


def _fit_head(arch, blob, proto_images, n_route):
    """Head weights and bias with which class c of the prototypes has logit 1 at output c % n_route and 0 elsewhere."""
    feat = _features(arch, blob, proto_images).double()
    p = feat.shape[0]
    want = torch.zeros((p, arch.n_classes), dtype=torch.float64, device="cuda")
    want[torch.arange(p), torch.arange(p) % n_route] = 1.0
    mu, ym = feat.mean(0), want.mean(0)
    d = feat - mu
    gram = d @ d.T
    gram += 1e-6 * gram.diagonal().mean() * torch.eye(p, device="cuda")
    w = (torch.linalg.solve(gram, want - ym).T @ d).float()
    specs, _ = W.blob_layout(arch)
    sw, sb = [s for s in specs if s.layer == arch.n_layers - 1 and s.name in ("w", "b")]
    w = w.to(torch.bfloat16) if arch.dtype == W.DT_BF16 else w
    blob[sw.offset:sw.offset + sw.nbytes] = w.flatten().contiguous().view(torch.uint8)
    blob[sb.offset:sb.offset + sb.nbytes] = (ym - w.double() @ mu).float().view(torch.uint8)


# ---- a case ----------------------------------------------------------------------------------------------------
def prepare(case, seed):
    gen = torch.Generator(device="cuda")
    gen.manual_seed(seed)
    n = case["n"]
    if case["kind"] == "regroup":
        e = case["experts"]
        rng = np.random.default_rng([seed, 2])
        cur = np.where(rng.random(n) < case["live"], rng.choice(e, size=n, p=W.zipf_probs(e, 1.1)), -1).astype(np.int32)
        out = [torch.full((m,), -1, dtype=torch.int32, device="cuda") for m in (e, e + 1, n, n)]      # cnt, off, perm, inv
        return dict(kind="regroup", n=n, experts=e, cur=torch.from_numpy(cur).cuda(), out=out)

    archs, e_arch, lists, prob, first_prob, class_prob = _model(case)
    rng = np.random.default_rng([seed, 1])
    fan, hw = len(class_prob), case["hw"]
    cls = rng.choice(fan, size=n, p=class_prob)
    first = rng.choice(len(first_prob), size=n, p=first_prob).astype(np.int32) if len(first_prob) > 1 else None
    proto = torch.randn((fan, GRID, GRID, 3), generator=gen, device="cuda")
    x = _images(proto, torch.from_numpy(cls).cuda(), hw, gen)
    exemplars = _images(proto, torch.arange(fan, device="cuda"), hw, gen)
    if case["kind"] == "tiny":
        x, exemplars = x.float(), exemplars.float()
    blobs = []
    for e, succ in enumerate(lists):
        blob = _blob(archs[e_arch[e]], gen)
        if succ:
            _fit_head(archs[e_arch[e]], blob, exemplars, len(succ))
        blobs.append(blob.cpu().numpy())

    # the schedules that the benchmark runs these kinds of workloads with
    tree50, vit = case["kind"] == "tree50", case["kind"] == "vit"
    stages = STAGES[case["kind"]]
    ctx = B.Context(max_requests=n, max_stages=stages, max_batch=512 if tree50 or vit else 4096, cache_cap_experts=case.get("cap", 0),
                    group_small=0 if tree50 or vit else 512, prefetch_depth=4 if tree50 else 2 if vit else 0, executors=3 if tree50 else 1)
    ids = [ctx.coe_register_arch(a) for a in archs]
    for e, blob in enumerate(blobs):
        ctx.coe_register_expert(e, ids[e_arch[e]], blob, prob[e])
    g = W.graph_from_lists(lists)
    ctx.coe_set_dependency_graph(g.succ_off, g.succ)
    if tree50:
        ctx.coe_set_latency_model(ids[0], 14000, 1600000, 850000)
        ctx.coe_set_arranging(ids[0], 0, 43, 8)
    host = case.get("host", False)
    if host:
        x = x.view(torch.int16).cpu().numpy().view(np.uint16)
    torch.cuda.synchronize()
    return dict(kind=case["kind"], n=n, ctx=ctx, x=x, first=first, host=host, arrival=case.get("arrival", n), stages=stages,
                window=tree50)


def run(state):
    n = state["n"]
    if state["kind"] == "regroup":
        cnt, off, perm, inv = state["out"]
        B.coe_regroup_static(n, state["cur"].data_ptr(), state["experts"], cnt.data_ptr(), off.data_ptr(), perm.data_ptr(), inv.data_ptr(),
                             torch.cuda.current_stream().cuda_stream)
        return cnt, off, perm, inv
    ctx, x, first = state["ctx"], state["x"], state["first"]
    for s in range(0, n, state["arrival"]):
        m = min(state["arrival"], n - s)
        images = x[s:s + m] if state["host"] else x[s].data_ptr()
        ctx.coe_submit(m, images, not state["host"], None if first is None else first[s:s + m])
        ctx.coe_step()
    if state["window"]:                       # groups may wait for later arrivals: step until the queue is empty
        while ctx.coe_step()[0] != B.COE_DONE:
            pass
    else:
        for _ in range(state["stages"] - 1):
            ctx.coe_step()
    _, logits, path = ctx.coe_collect(n)
    return logits, path


def _macs(arch):
    """Multiply-accumulates of one request."""
    total = 0
    for layer, ((h, w, c), d) in zip(arch.layers, W.walk(arch)):
        op, k, r, s = int(layer[0]), int(layer[4]), int(layer[5]), int(layer[6])
        if op == W.OP_CONV:
            total += d[0] * d[1] * k * r * s * c
        elif op in (W.OP_HEAD, W.OP_HEAD_CLS):
            total += k * c
        elif op == W.OP_ATTENTION:
            total += 2 * h * w * h * w * (c // 3)
    return total


def work(case):
    n = case["n"]
    if case["kind"] == "regroup":
        # keys in; counts, offsets, permutation and inverse out
        return {"bytes": 4 * n + 4 * (2 * case["experts"] + 1) + 4 * n + 4 * int(case["live"] * n), "flops": 0}
    archs, e_arch, _, prob, _, _ = _model(case)
    # the expected visits of every expert; an expert's weights are read once if a request reaches it
    visits = [n * p for p in prob]
    macs = [_macs(a) for a in archs]
    size = [W.blob_layout(a)[1] for a in archs]
    flops = sum(2.0 * visits[e] * macs[a] for e, a in enumerate(e_arch))
    weights = sum(min(1.0, visits[e]) * size[a] for e, a in enumerate(e_arch))
    row = archs[0].input_elems * archs[0].elem_bytes
    out = 4 * max(a.n_classes for a in archs) + 4 * STAGES[case["kind"]]
    return {"bytes": int(n * (row + out) + weights), "flops": int(flops)}


def tolerance(case):
    # about four times the distance of the logits from the oracle's, which stores the same roundings but sums in 64 bits
    # (measured: ResNet- and mixed shapes 0.9e-3 to 1.5e-3 on 224 x 224 images and 3.1e-3 on 64 x 64, whose pooled
    # features average fewer pixels; detectors 2.0e-3; the deeper transformers 8.7e-3 to 9.1e-3; fp32 experts 2.2e-7)
    if case["kind"] == "regroup":
        return "exact"
    if case["kind"] == "tiny":
        return {"rel": 1e-6}
    if case["kind"] == "vit":
        return {"rel": 3.5e-2}
    return {"rel": 6e-3 if case["hw"] >= 192 else 1.2e-2}
