"""Performance cases of the dense-block library: what a user of it has it do, through the calls of
`paper_1707_06990_amd` (the C ABI's names), over the range of sizes it serves.

A case is a dict of plain values.  "kind" is one of
  net    a CIFAR-shaped DenseNet-BC training step, fp32 NCHW        (dnb_net_forward / _backward)
  inet   an ImageNet-shaped DenseNet-BC training step, bf16 NHWC    (dnb_inet_forward / _backward)
  block  one dense block, fp32 NCHW or bf16 NHWC                    (dnb_block_forward / _backward)
and "direction" is "step" (forward and backward) or "forward".  Calls are made one after the other
on the current stream, as a training loop makes them; with "graph" the step is captured once, when
the state is made, and a pass replays it.
"""
import functools
import math

import numpy as np
import torch

import paper_1707_06990_amd as dnb

SCHEDULES = {"shared": dnb.DNB_SCHED_SHARED, "store_all": dnb.DNB_SCHED_STORE_ALL, "fused": dnb.DNB_SCHED_FUSED}


def _net(name, n, image, depth, growth, classes, schedule="fused", direction="step", graph=False):
    return {"name": name, "kind": "net", "n": n, "image": image, "depth": depth, "growth": growth, "classes": classes,
            "schedule": schedule, "direction": direction, "graph": graph}


def _inet(name, n, image, growth, layers, classes, schedule="fused", direction="step", graph=False):
    return {"name": name, "kind": "inet", "n": n, "image": image, "growth": growth, "m0": layers[0], "m1": layers[1],
            "m2": layers[2], "m3": layers[3], "classes": classes, "schedule": schedule, "direction": direction,
            "graph": graph}


def _block(name, dtype, n, c0, h, w, layers, growth, bottleneck, schedule="fused", direction="step", graph=False):
    return {"name": name, "kind": "block", "dtype": dtype, "n": n, "c0": c0, "h": h, "w": w, "layers": layers,
            "growth": growth, "bottleneck": bottleneck, "schedule": schedule, "direction": direction, "graph": graph}


def listed():
    return [
        # the benchmark's smallest workload: one small block, where launches and latency are all there is
        _block("block_small", "f32", 2, 16, 8, 8, 4, 12, 48),
        # the headline workload, as a loop that calls the library step by step runs it
        _net("bc100_step", 64, 32, 100, 12, 10),
        # ... and captured once in a HIP graph and replayed, as the benchmark and a tuned loop run it
        _net("bc100_graph", 64, 32, 100, 12, 10, graph=True),
        # the same network under the paper's own schedule (shared storages filled and re-filled)
        _net("bc100_shared", 64, 32, 100, 12, 10, schedule="shared"),
        # the deep and wide fp32 network: matrix-bound layers, up to 2000 input channels
        _net("bc250_step", 64, 32, 250, 24, 100),
        # odd batch and an image size whose blocks are 28x28, 14x14 and 7x7 (rows not a multiple of
        # 16 bytes), a last batch of an epoch: what the any-shape kernels have to take
        _net("bc40_ragged", 37, 28, 40, 12, 10, schedule="shared"),
        # a dense block without bottleneck, the first form the paper gives: the second block of the
        # L = 40, k = 12 network (12 layers, 160 channels in, 16x16)
        _block("plain_block", "f32", 64, 160, 16, 16, 12, 12, 0, schedule="shared"),
        # the two ImageNet-shaped training steps
        _inet("dn161_step", 32, 224, 48, (6, 12, 36, 24), 1000),
        _inet("dn264_step", 32, 224, 32, (6, 12, 64, 48), 1000),
        # a small batch through the large network (fine-tuning, a debug run): short kernels, long chains
        _inet("dn161_batch2", 2, 224, 48, (6, 12, 36, 24), 1000),
        # forward only (computing features and losses without training on them)
        _inet("dn264_forward", 32, 224, 32, (6, 12, 64, 48), 1000, direction="forward"),
        # one bf16 block under the paper's schedule, 28x28, an odd batch
        _block("bf16_block_shared", "bf16", 17, 256, 28, 28, 12, 32, 128, schedule="shared"),
    ]


def _log_int(rng, lo, hi, step=1):
    v = math.exp(rng.uniform(math.log(lo), math.log(hi)))
    return max(lo, min(hi, int(round(v / step)) * step))


def draw(rng):
    """One more case of the same ranges: the kinds above with sizes spread over what they stand for."""
    kind = rng.choice(["net", "net", "inet", "inet", "block", "block", "plain", "bf16_block"])
    direction = rng.choice(["step", "step", "step", "forward"])
    while True:
        if kind == "net":
            image = rng.choice([16, 24, 28, 32, 32, 40, 48])
            schedule = "shared" if image % 16 else rng.choice(["fused", "fused", "shared", "store_all"])
            c = _net("", _log_int(rng, 2, 128), image, 6 * rng.randint(2, 30) + 4, rng.choice([8, 12, 12, 16, 24, 24, 32]),
                     rng.choice([10, 100]), schedule, direction, graph=rng.random() < 0.2)
        elif kind == "inet":
            growth = rng.choice([16, 32, 32, 48])
            layers = (rng.randint(2, 6), rng.randint(2, 12), rng.randint(4, 64), rng.randint(2, 48))
            c = _inet("", _log_int(rng, 1, 48), rng.choice([96, 160, 224, 224, 256]), growth, layers,
                      rng.choice([100, 1000]), rng.choice(["fused", "fused", "fused", "shared"]), direction)
        elif kind == "block":
            k = rng.choice([8, 12, 12, 16, 24, 32])
            w = rng.choice([8, 12, 16, 20, 32, 9, 14, 28])
            schedule = rng.choice(["fused", "fused", "shared", "store_all"]) if w % 4 == 0 else "shared"
            c = _block("", "f32", _log_int(rng, 1, 96), rng.randint(8, 300), rng.choice([w, w, w + 3]), w,
                       rng.randint(1, 24), k, 4 * k, schedule, direction)
        elif kind == "plain":
            w = rng.choice([8, 14, 16, 32])
            c = _block("", "f32", _log_int(rng, 1, 64), _log_int(rng, 3, 200), w, w, rng.randint(2, 12), rng.choice([8, 12, 16]),
                       0, rng.choice(["shared", "store_all"]), direction)
        else:
            k = rng.choice([16, 32, 48])
            w = rng.choice([7, 12, 14, 28, 40, 56])
            c = _block("", "bf16", _log_int(rng, 1, 48), 8 * rng.randint(2, 100), w, w, rng.randint(1, 24), k, 4 * k,
                       rng.choice(["fused", "fused", "shared", "store_all"]), direction)
        del c["name"]
        # no more than the largest listed case; less where the any-shape kernels take it, which are
        # far slower per operation
        most, mine = work(_net("", 64, 32, 250, 24, 100)), work(c)
        odd = kind == "plain" or c.get("w", c.get("image")) % 16 != 0
        share = 1.0 if c["schedule"] == "fused" else 0.03 if odd else 0.2
        if mine["flops"] <= share * most["flops"] and mine["bytes"] <= most["bytes"] and _create_ok(c):
            return c


# ---------------------------------------------------------------- shapes

def _blocks_of(case):
    """(n, c0, h, w, layers, growth, bottleneck) of every dense block of a case."""
    if case["kind"] == "block":
        return [tuple(case[k] for k in ("n", "c0", "h", "w", "layers", "growth", "bottleneck"))]
    k = case["growth"]
    if case["kind"] == "net":
        c, s, ms = 2 * k, case["image"], [(case["depth"] - 4) // 6] * 3
    else:
        c, s, ms = 2 * k, case["image"] // 4, [case["m%d" % i] for i in range(4)]
    out = []
    for m in ms:
        out.append((case["n"], c, s, s, m, k, 4 * k))
        c = (c + m * k) // 2
        s //= 2
    return out


class _Handle:
    """A library handle that is destroyed with the state that holds it."""

    def __init__(self, h, destroy):
        self.h, self.destroy = h, destroy

    def __del__(self):
        self.destroy(self.h)


def _create(case):
    sched = SCHEDULES[case["schedule"]]
    if case["kind"] == "net":
        return _Handle(dnb.dnb_net_create(case["n"], case["image"], case["depth"], case["growth"], case["classes"],
                                          schedule=sched), dnb.dnb_net_destroy)
    if case["kind"] == "inet":
        return _Handle(dnb.dnb_inet_create(case["n"], case["image"], case["growth"], [case["m%d" % i] for i in range(4)],
                                           case["classes"], schedule=sched), dnb.dnb_inet_destroy)
    bf16 = case["dtype"] == "bf16"
    return _Handle(dnb.dnb_block_create(*_blocks_of(case)[0], dtype=dnb.DNB_BF16 if bf16 else dnb.DNB_F32,
                                        layout=dnb.DNB_NHWC if bf16 else dnb.DNB_NCHW, schedule=sched),
                   dnb.dnb_block_destroy)


def _create_ok(case):
    try:
        _create(case)
        return True
    except dnb.DnbError:
        return False


def _parts(case, h):
    """The parameter pack as a list of (name, offset, count, kind, fan_in), kind g | b | W | 0."""
    out = []

    def block(base, c0, m, k, B, tag):
        o = base
        for l in range(m):
            c = c0 + l * k
            shapes = ([("g", c, 0), ("b", c, 0), ("W", B * c, c), ("g", B, 0), ("b", B, 0), ("W", k * B * 9, 9 * B)]
                      if B else [("g", c, 0), ("b", c, 0), ("W", k * c * 9, 9 * c)])
            for kind, cnt, fan in shapes:
                out.append((tag, o, cnt, kind, fan))
                o += cnt
        return o - base

    bl = _blocks_of(case)
    if case["kind"] == "block":
        n = block(0, bl[0][1], bl[0][4], bl[0][5], bl[0][6], "block")
        assert n == dnb.dnb_block_param_count(h)
        return out
    k, classes = case["growth"], case["classes"]
    if case["kind"] == "net":
        offset = lambda p: dnb.dnb_net_param_offset(h, p)
        P = dnb
        out.append(("stem", *offset(P.DNB_NP_STEM), "W", 27))
        bparts = [P.DNB_NP_BLOCK0 + b for b in range(3)]
        after = [(P.DNB_NP_TRANS0_G, P.DNB_NP_TRANS0_B, P.DNB_NP_TRANS0_W),
                 (P.DNB_NP_TRANS1_G, P.DNB_NP_TRANS1_B, P.DNB_NP_TRANS1_W),
                 (P.DNB_NP_TAIL_G, P.DNB_NP_TAIL_B, P.DNB_NP_TAIL_WL)]
        bias = P.DNB_NP_TAIL_BL
    else:
        offset = lambda p: dnb.dnb_inet_param_offset(h, p)
        P = dnb
        out.append(("stem", *offset(P.DNB_IP_STEM_W), "W", 147))
        out.append(("stem", *offset(P.DNB_IP_STEM_G), "g", 0))
        out.append(("stem", *offset(P.DNB_IP_STEM_B), "b", 0))
        bparts = [P.DNB_IP_BLOCK0 + 4 * b for b in range(4)]
        after = [tuple(P.DNB_IP_BLOCK0 + 4 * b + i for i in (1, 2, 3)) for b in range(4)]
        bias = P.DNB_IP_TAIL_BL
    for b, (_, c0, _, _, m, kk, B) in enumerate(bl):
        off, cnt = offset(bparts[b])
        assert block(off, c0, m, kk, B, "block%d" % b) == cnt
        c = c0 + m * kk
        tag = "trans%d" % b if b + 1 < len(bl) else "tail"
        for p, kind in zip(after[b], "gbW"):
            out.append((tag, *offset(p), kind, c))
    out.append(("tail", *offset(bias), "0", 0))
    return out


@functools.lru_cache(maxsize=4)
def _pack_recipe(key):
    """(std, mean) per parameter and the named ranges of the pack, for a case given as sorted items."""
    case = dict(key)
    hd = _create(case)
    parts = _parts(case, hd.h)
    total = max(o + c for _, o, c, _, _ in parts)
    std, mean = np.zeros(total, np.float32), np.zeros(total, np.float32)
    ranges = {}
    for tag, o, c, kind, fan in parts:
        # He-normal weights; BN scales around one and shifts around zero, as in a network being trained
        std[o:o + c] = {"W": math.sqrt(2.0 / fan) if fan else 0.0, "g": 0.25, "b": 0.25, "0": 0.0}[kind]
        mean[o:o + c] = 1.0 if kind == "g" else 0.0
        lo, hi = ranges.get(tag, (o, o + c))
        ranges[tag] = (min(lo, o), max(hi, o + c))
    return std, mean, ranges


# ---------------------------------------------------------------- the measured path

def prepare(case, seed):
    case = {k: v for k, v in case.items() if k != "name"}
    gen = torch.Generator(device="cuda").manual_seed(int(seed))
    rand = lambda *shape: torch.randn(*shape, device="cuda", generator=gen)
    std, mean, ranges = _pack_recipe(tuple(sorted(case.items())))
    handle = _create(case)
    h = handle.h
    st = {"case": case, "handle": handle}
    st["params"] = rand(std.size).mul_(torch.from_numpy(std).cuda()).add_(torch.from_numpy(mean).cuda())
    st["dparams"] = torch.empty_like(st["params"])
    st["grads"] = {tag: st["dparams"][lo:hi] for tag, (lo, hi) in ranges.items()}
    n = case["n"]
    if case["kind"] == "block":
        bf16 = case["dtype"] == "bf16"
        dt = torch.bfloat16 if bf16 else torch.float32
        c_out = case["c0"] + case["layers"] * case["growth"]
        shape = (lambda c: (n, case["h"], case["w"], c)) if bf16 else (lambda c: (n, c, case["h"], case["w"]))
        st["x0"], st["dy"] = rand(*shape(case["c0"])).to(dt), rand(*shape(c_out)).to(dt)
        st["y"], st["dx0"] = torch.empty_like(st["dy"]), torch.empty_like(st["x0"])
        nbytes = dnb.dnb_block_workspace_bytes(h)
    else:
        image = case["image"]
        if case["kind"] == "net":
            st["x"] = rand(n, 3, image, image)
            nbytes = dnb.dnb_net_workspace_bytes(h)
        else:
            st["x"] = rand(n, image, image, 3).to(torch.bfloat16)
            nbytes = dnb.dnb_inet_workspace_bytes(h)
        st["labels"] = torch.randint(0, case["classes"], (n,), device="cuda", generator=gen, dtype=torch.int32)
        st["loss"] = torch.empty(1, device="cuda")
        st["logits"] = torch.empty(n, case["classes"], device="cuda")
    st["ws"] = torch.empty(nbytes, dtype=torch.uint8, device="cuda")
    if case["graph"]:
        side = torch.cuda.Stream()
        side.wait_stream(torch.cuda.current_stream())
        with torch.cuda.stream(side):
            _call(st)
        torch.cuda.current_stream().wait_stream(side)
        graph = torch.cuda.CUDAGraph()
        with torch.cuda.graph(graph):
            _call(st)
        st["graph"] = graph
    return st


def _call(st):
    """The forward and backward calls of one pass, on the current stream."""
    case, h = st["case"], st["handle"].h
    if case["kind"] == "block":
        dnb.dnb_block_forward(h, st["x0"], st["params"], st["y"], st["ws"])
        if case["direction"] == "step":
            dnb.dnb_block_backward(h, st["params"], st["y"], st["dy"], st["dx0"], st["dparams"], st["ws"])
    elif case["kind"] == "net":
        dnb.dnb_net_forward(h, st["x"], st["labels"], st["params"], st["loss"], st["logits"], st["ws"])
        if case["direction"] == "step":
            dnb.dnb_net_backward(h, st["x"], st["params"], st["dparams"], st["ws"])
    else:
        dnb.dnb_inet_forward(h, st["x"], st["labels"], st["params"], st["loss"], st["logits"], st["ws"])
        if case["direction"] == "step":
            dnb.dnb_inet_backward(h, st["x"], st["params"], st["dparams"], st["ws"])


def run(st):
    if "graph" in st:
        st["graph"].replay()
    else:
        _call(st)
    out = {"y": st["y"]} if st["case"]["kind"] == "block" else {"loss": st["loss"], "logits": st["logits"]}
    if st["case"]["direction"] == "step":
        if st["case"]["kind"] == "block":
            out["dx0"] = st["dx0"]
        out["dparams"] = st["grads"]
    return out


# ---------------------------------------------------------------- what a pass cannot do without

def work(case):
    """Bytes: inputs, parameters and outputs once, and the feature maps that the method keeps from
    forward to backward (every conv output) written once and, in a step, read once.  Flops: the
    convolutions' products, three times (output, data gradient, weight gradient) in a step."""
    step = case["direction"] == "step"
    esz = 2 if case["kind"] == "inet" or case.get("dtype") == "bf16" else 4
    flops = kept = params = 0
    bl = _blocks_of(case)
    for i, (n, c0, h, w, m, k, B) in enumerate(bl):
        P = n * h * w
        for l in range(m):
            c = c0 + l * k
            flops += 2 * P * (c * B + 9 * B * k if B else 9 * c * k)
            params += 2 * c + (B * c + 2 * B + 9 * k * B if B else 9 * k * c)
        kept += P * (c0 + m * (k + B)) * esz
        if case["kind"] != "block" and i + 1 < len(bl):
            c = c0 + m * k
            flops += 2 * P * c * (c // 2)
            params += 2 * c + c * (c // 2)
    if case["kind"] == "block":
        n, c0, h, w, m, k, B = bl[0]
        io = n * h * w * esz * (c0 + ((c0 + m * k) + c0 if step else 0))
    else:
        ks, so = (3, case["image"]) if case["kind"] == "net" else (7, case["image"] // 2)
        flops += 2 * case["n"] * so * so * 2 * case["growth"] * 3 * ks * ks
        c = bl[-1][1] + bl[-1][4] * bl[-1][5]
        flops += 2 * case["n"] * c * case["classes"]
        params += 2 * case["growth"] * 3 * ks * ks + c * case["classes"]
        io = case["n"] * 3 * case["image"] ** 2 * esz
    return {"bytes": int(io + (2 if step else 1) * (kept + 4 * params)), "flops": int((3 if step else 1) * flops)}


def tolerance(case):
    """What another correct implementation at the same precision would show (2-norm, per output).

    Measured by moving every parameter by about half a unit in the last place of fp32, which moves
    results as another order of the sums does.  fp32 forward: 2e-6 of the logits and of y, more
    where a chain adds thousands of products.  fp32 gradients: 6e-3 in the deepest network: among
    some 1e8 ReLU decisions a few lie within rounding of zero, and each that falls the other way
    moves gradient elements by their whole size.  bf16: a feature rounded the other way moves by
    2^-8, so the logits of the deep networks move by 2e-2; their gradients, if that happens in the
    forward pass, move by far more than any bound says (ReLU decisions on bf16 features), so a bf16
    step is held to the most that can be stated, and with it to the forward pass's own roundings."""
    bf16 = case["kind"] == "inet" or case.get("dtype") == "bf16"
    if bf16:
        return {"rel": 0.03, "max": 0.95}
    if case["direction"] == "forward":
        return {"rel": 3e-5, "max": 1e-3}
    return {"rel": 0.02, "max": 0.95}
