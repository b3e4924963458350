"""The work a user of this framework has it do, as timed cases through the public entry points.

Every case is one pass of the online phase: the offline material (triples, masks, prepared planes, folded addends)
and the weights are what a program holds before a batch arrives, the input shares are the batch.  Lanes run as the
benchmark's step runs them (one in-order queue, exchange by remote store, folded prepared linear layers,
preallocated outputs) unless a case says otherwise.  All results are ring words and compared exactly.
"""
import math

import torch

from paper_2209_13643_amd import dealer, mpc, pipeline, synth

DEVICE = "cuda:0"
MAX_MACS = 4096 * 768 * 3072          # the largest single layer listed
MAX_WORDS = 32 * 56 * 56 * 256        # words of the largest activation listed


def listed():
    return [
        # the first thing a user runs: a dense layer of 64 rows and its ReLU on a lane made with the defaults
        # (three streams, copy exchange); all latency and launches
        dict(name="tiny-layer", kind="layer", M=64, K=256, N=128),
        # ReLU behind a small layer (the 512-wide head, 32 images per micro-batch, plus a ragged tail)
        dict(name="relu-16k-odd", kind="relu", n=16411, packed=False),
        # ReLU of the VGG-style block at batch 64, whole-word adder and sign-only chain
        dict(name="relu-2m", kind="relu", n=64 * 16 * 16 * 128, packed=False),
        dict(name="relu-sign-2m", kind="relu", n=64 * 16 * 16 * 128, packed=True),
        # the VGG-style 3x3 block
        dict(name="conv-3x3-128", kind="conv", B=64, HW=16, Cin=128, Cout=128, k=3, stride=1),
        # the bottleneck's widening 1x1 convolution: short contraction, the largest activations
        dict(name="conv-1x1-64-256", kind="conv", B=32, HW=56, Cin=64, Cout=256, k=1, stride=1),
        # encoder feed-forward, and one head of the ImageNet classifier at two images (few rows, large weights)
        dict(name="dense-ffn1", kind="dense", M=4096, K=768, N=3072),
        dict(name="dense-fc-2rows", kind="dense", M=2, K=25088, N=4096),
        # per-head Q K^T: a product of two activations
        dict(name="attention-qk", kind="attention", heads=96, T=512, dh=64, product="qk"),
        # the headline: VGG16 on 32x32 images, batch 128 as four micro-batches on four lanes
        dict(name="vgg16-forward", kind="network", mb=4, batch=32, packed=False),
        # a training step (forward with tape, backward, all weight gradients) of one micro-batch
        dict(name="vgg16-train", kind="train", batch=32, packed=True),
        # the VGG-style block with three parties: convolution, masked rescale, ReLU
        dict(name="block-3-parties", kind="layer3", B=64, HW=16, Cin=128, Cout=128, packed=False),
    ]


def _log(rng, lo, hi):
    return max(lo, min(hi, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


def draw(rng):
    kind = rng.choice(["layer", "relu", "relu", "conv", "conv", "dense", "dense", "attention", "network", "train", "layer3"])
    if kind == "layer":
        return dict(kind=kind, M=_log(rng, 1, 512), K=_log(rng, 16, 1024), N=_log(rng, 8, 512))
    if kind == "relu":
        return dict(kind=kind, n=_log(rng, 1000, 4 << 20), packed=rng.random() < 0.5)
    if kind == "conv":
        while True:
            k = rng.choice([1, 3, 3])
            c = dict(kind=kind, B=_log(rng, 1, 64), HW=rng.randint(7, 56), Cin=_log(rng, 3, 512), Cout=_log(rng, 16, 512), k=k,
                     stride=rng.choice([1, 1, 1, 2]))
            px = c["B"] * c["HW"] ** 2
            if px * max(c["Cin"], c["Cout"]) <= MAX_WORDS and px * k * k * c["Cin"] * c["Cout"] <= MAX_MACS:
                return c
    if kind == "dense":
        while True:
            c = dict(kind=kind, M=_log(rng, 1, 4096), K=_log(rng, 64, 25088), N=_log(rng, 10, 4096))
            if c["M"] * c["K"] * c["N"] <= MAX_MACS and c["K"] * c["N"] <= 25088 * 4096:
                return c
    if kind == "attention":
        return dict(kind=kind, heads=_log(rng, 1, 96), T=_log(rng, 16, 512), dh=64, product=rng.choice(["qk", "av"]))
    if kind == "network":
        return dict(kind=kind, mb=rng.randint(1, 4), batch=_log(rng, 1, 32), packed=rng.random() < 0.5)
    if kind == "train":
        return dict(kind=kind, batch=_log(rng, 1, 32), packed=rng.random() < 0.5)
    return dict(kind=kind, B=_log(rng, 1, 64), HW=rng.choice([4, 7, 8, 14, 16]), Cin=_log(rng, 16, 128), Cout=_log(rng, 16, 128),
                packed=rng.random() < 0.5)


# ------------------------------------------------------------------------------------------------ states
def _lane(exchange="put"):
    ln = mpc.Lane(0, single_queue=True)
    ln.set_exchange(exchange)
    return ln


def _pair(shape, n=2):
    return tuple(torch.empty(shape, dtype=torch.int64, device=DEVICE) for _ in range(n))


def _conv(c):
    return synth.Conv("conv", c["B"], c["HW"], c["HW"], c["Cin"], c["Cout"], c["k"], c["k"], c["k"] // 2, c["stride"],
                      1.0, synth.he_std(c["k"] * c["k"] * c["Cin"]))


def _vgg(c):
    return pipeline.with_batch(synth.config_vgg16_pipeline().layers, c["batch"])


def _state_of(d):
    return pipeline.LayerState(w=d["w"], a=d["a"], b=d["b"], c=d["c"], f_public=d["f_public"])


def prepare(case, seed):
    g = dealer.gen(seed, DEVICE)
    kind = case["kind"]
    s = dict(kind=kind)
    if kind == "layer":
        ln = mpc.Lane(0)
        M, K, N = case["M"], case["K"], case["N"]
        d = dealer.matmul_layer(ln, g, M, K, N, 1.0, K ** -0.5)
        s.update(lane=ln, d=d, mat=dealer.relu_material(g, M * N, DEVICE), z=_pair((M, N)), y=_pair((M, N)))
        ln.reserve(max(mpc.lib().mpc_matmul_workspace_bytes(M, K, N, 1), mpc.lib().mpc_relu_workspace_bytes(M * N)))
    elif kind == "relu":
        n = case["n"]
        x = dealer.share(g, dealer.normal_fixed(g, (n,), 1.0, DEVICE))
        s.update(lane=_lane(), x=x, mat=dealer.relu_material(g, n, DEVICE, packed=case["packed"]), packed=case["packed"], y=_pair((n,)))
    elif kind in ("conv", "dense"):
        ln = _lane()
        if kind == "conv":
            L = _conv(case)
            d = dealer.conv_layer(ln, g, L.B, L.H, L.W, L.Cin, L.Cout, L.KH, L.KW, L.pad, L.stride, L.x_std, L.w_std)
        else:
            L = synth.Gemm("dense", case["M"], case["K"], case["N"], 1.0, synth.he_std(case["K"]))
            d = dealer.matmul_layer(ln, g, L.M, L.K, L.N, L.x_std, L.w_std)
        st = _state_of(d)
        pipeline.prepare_layers(ln, [L], [st], fold=True)
        s.update(lane=ln, L=L, st=st, x=d["x"], out=pipeline.alloc_outputs(ln, [L], [st])[0])
    elif kind == "attention":
        ln = _lane()
        H, T, dh = case["heads"], case["T"], case["dh"]
        M, K, N = (T, dh, T) if case["product"] == "qk" else (T, T, dh)
        d = dealer.matmul_layer(ln, g, M, K, N, 1.0, 1.0, batch=H)
        right, left = ln.prepare_matmul(d["a"], d["b"], None)
        c_fold = (ln.fold_matmul(d["a"], d["b"], d["c"]), d["c"][1])
        s.update(lane=ln, d=d, right=right, left=left, c=c_fold, z=_pair((H, M, N)))
        ln.sync()
    elif kind == "network":
        layers = _vgg(case)
        lanes = [_lane() for _ in range(case["mb"])]
        weights = pipeline.deal_weights(g, layers, DEVICE)
        states, xs, outs = [], [], []
        for ln in lanes:
            st = pipeline.deal_microbatch(ln, g, layers, weights, packed_relu=case["packed"])
            pipeline.prepare_layers(ln, layers, st, fold=True)
            L = layers[0]
            xs.append(dealer.share(g, dealer.normal_fixed(g, (L.B, L.H, L.W, L.Cin), 1.0, DEVICE)))
            states.append(st); outs.append(pipeline.alloc_outputs(ln, layers, st))
        s.update(lanes=lanes, layers=layers, states=states, xs=xs, outs=outs)
    elif kind == "train":
        layers = _vgg(case)
        ln = _lane()
        weights = pipeline.deal_weights(g, layers, DEVICE)
        st = pipeline.deal_microbatch(ln, g, layers, weights, packed_relu=case["packed"])
        pipeline.preopen_weights(ln, st)
        bst = pipeline.deal_backward(ln, g, layers, st)
        L = layers[0]
        x = dealer.share(g, dealer.normal_fixed(g, (L.B, L.H, L.W, L.Cin), 1.0, DEVICE))
        gout = dealer.share(g, dealer.normal_fixed(g, (layers[-1].M, layers[-1].N), 0.5, DEVICE))
        s.update(lane=ln, layers=layers, st=st, bst=bst, x=x, gout=gout)
    elif kind == "layer3":
        ln = _lane()
        B, HW, Cin, Cout = case["B"], case["HW"], case["Cin"], case["Cout"]
        d = dealer.conv_layer3(ln, g, B, HW, HW, Cin, Cout, 3, 3, 1, 1, 1.0, synth.he_std(9 * Cin))
        mat = dealer.relu3_material(g, B * HW * HW * Cout, DEVICE, packed=case["packed"])
        f_public = ln.open3(ln.sub3(d["w"], d["b"]))
        right, left = ln.prepare_conv2d3(d["a"], d["b"], f_public, 1, 1)
        ln.sync()
        s.update(lane=ln, d=d, mat=mat, right=right, left=left, packed=case["packed"],
                 z=_pair((B, HW, HW, Cout), 3), y=_pair((B, HW, HW, Cout), 3))
    else:
        raise ValueError(kind)
    torch.cuda.synchronize()
    return s


# ------------------------------------------------------------------------------------------------ passes
def run(s):
    kind = s["kind"]
    if kind == "layer":
        ln, d = s["lane"], s["d"]
        ln.beaver_matmul(d["x"], d["w"], d["a"], d["b"], d["c"], out=s["z"])
        return s["z"], ln.relu(s["z"], s["mat"], out=s["y"])
    if kind == "relu":
        return s["lane"].relu(s["x"], s["mat"], packed=s["packed"], out=s["y"])
    if kind in ("conv", "dense"):
        return pipeline.run_layer(s["lane"], s["L"], s["st"], s["x"], [], out=s["out"])
    if kind == "attention":
        d = s["d"]
        return s["lane"].beaver_matmul_folded(d["x"], d["w"], d["a"], d["b"], s["c"], s["right"], s["left"], out=s["z"])
    if kind == "network":
        return pipeline.forward_pipelined(s["lanes"], s["layers"], s["states"], s["xs"], [], outs_per_mb=s["outs"])
    if kind == "train":
        keep = []
        logits, tape = pipeline.forward_train(s["lane"], s["layers"], s["st"], s["x"], keep)
        grads = pipeline.backward(s["lane"], s["layers"], s["st"], s["bst"], tape, s["gout"], keep)
        s["lane"].sync()              # the tape and the kept intermediates go when the step is done
        return logits, grads
    ln, d = s["lane"], s["d"]
    z = ln.conv2d3_prepared(d["x"], d["a"], d["c"], s["right"], s["left"], 3, 3, 1, 1, out=s["z"])
    ln.truncate3(z, d["r"], d["rt"])
    return ln.relu3(z, s["mat"], out=s["y"], packed=s["packed"])


# ------------------------------------------------------------------------------------------------ work
W = 8
# int8 multiply-accumulates of one ring product mod 2^64: the bilinear rank of a product of eight digits mod x^8
RING_OPS = 2 * 15


def _relu_words(n, packed, parties=2):
    """Words of x, material and y of one secure ReLU, all parties, and bytes of its bit material."""
    triples = (13 if parties == 3 else 12)
    per = 3 * triples if not packed else 3 * (triples - 11) + 6 * 31 / 32 + 3 / 64
    return parties * n * (1 + (2 if parties == 3 else 1) + per + 1 + 3 + 1) * W + parties * n


def _linear(x, w, z, macs, products=3, parties=2):
    """x, a, c, z of every party, and the right operands (w's opened mask and the triple's b)."""
    return parties * (2 * x + 2 * z) * W + (parties + 1) * w * W, macs * products * RING_OPS


def _layer_work(L, packed, train):
    if isinstance(L, synth.Conv):
        M, K, N = L.gemm_mkn
        nx, nw = L.B * L.H * L.W * L.Cin, K * N
        pooled = L.B * (L.Ho // 2) * (L.Wo // 2) * L.Cout if L.pool else 0
    else:
        M, K, N, pooled = L.M, L.K, L.N, 0
        nx, nw = M * K, K * N
    nz = M * N
    by, fl = _linear(nx, nw, nz, M * K * N, 4 if train else 3)
    relu = _relu_words(nz, packed) if L.relu else 0
    pool = _relu_words(3 * pooled, packed)
    by += relu + pool
    if train:                          # both gradient products, element-wise products of ReLU and pooling
        by += 2 * (2 * (nx + nz) + 3 * nw) * W + 2 * (nx + nw) * W
        fl += 2 * M * K * N * 4 * RING_OPS
        by += 2 * 6 * ((nz if L.relu else 0) + 3 * pooled) * W
    return by, fl


def work(case):
    kind = case["kind"]
    if kind == "layer":
        M, K, N = case["M"], case["K"], case["N"]
        by, fl = _linear(M * K, K * N, M * N, M * K * N, 4)
        return {"bytes": by + _relu_words(M * N, False), "flops": fl}
    if kind == "relu":
        return {"bytes": _relu_words(case["n"], case["packed"]), "flops": 0}
    if kind == "conv":
        L = _conv(case)
        M, K, N = L.gemm_mkn
        by, fl = _linear(L.B * L.H * L.W * L.Cin, K * N, M * N, M * K * N)
        return {"bytes": by, "flops": fl}
    if kind == "dense":
        by, fl = _linear(case["M"] * case["K"], case["K"] * case["N"], case["M"] * case["N"], case["M"] * case["K"] * case["N"])
        return {"bytes": by, "flops": fl}
    if kind == "attention":
        H, T, dh = case["heads"], case["T"], case["dh"]
        nx, nw, nz = (T * dh, T * dh, T * T) if case["product"] == "qk" else (T * T, T * dh, T * dh)
        by, fl = _linear(H * nx, 0, H * nz, H * T * T * dh)
        return {"bytes": by + 4 * H * nw * W, "flops": fl}
    if kind in ("network", "train"):
        parts = [_layer_work(L, case["packed"], kind == "train") for L in _vgg(case)]
        mb = case.get("mb", 1)
        return {"bytes": mb * sum(p[0] for p in parts), "flops": mb * sum(p[1] for p in parts)}
    B, HW, Cin, Cout = case["B"], case["HW"], case["Cin"], case["Cout"]
    nz = B * HW * HW * Cout
    by, fl = _linear(B * HW * HW * Cin, 9 * Cin * Cout, nz, nz * 9 * Cin, 6, 3)
    return {"bytes": by + 3 * 2 * nz * W + _relu_words(nz, case["packed"], 3), "flops": fl}


def tolerance(case):
    return "exact"
