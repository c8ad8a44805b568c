"""Performance cases of the library: what programs that use it have it do, over the sizes they do it at.

Three kinds of program are covered, all through the entry points of include/bnn.h:

* a recogniser that scores frames with a trained network (``bnn_forward``), from one frame at a time on a device that
  listens, over single utterances, to large batches on a server;
* the same with the network families of the paper: binary activations in {-1, +1} or {0, 1}, real activations
  (hard-tanh), the mixed topology it recommends (Sigmoid in the first and last hidden layer, binary units between), the
  latter also with real-valued weights in the input and the Softmax layer;
* a training step (Alg. 1 and Alg. 2): binarise, forward with the pre-activations kept, backward, update.

Network shapes are those of workloads/synth.py (440 inputs, 3 to 6 hidden layers of 512 to 4096 units, 1000 to 4000
tied states) and others between them; ``draw`` spreads widths, outputs and frames over the same ranges, ragged sizes
among them.  Weights are uniform on (-1, 1), inputs and biases normal, as in workloads/synth.py, made on the GPU.
"""
from __future__ import annotations

import math

import torch

import paper_1706_09453_amd as bnn

DEV = "cuda:0"

SIGN, STEP01, HARDTANH, MIXED = "sign", "step01", "hardtanh", "mixed"


def _forward(name, frames, hidden, layers, outputs, act, word_bits=32, real_io=False, inputs=440):
    return {"name": name, "kind": "forward", "frames": frames, "inputs": inputs, "hidden": hidden, "layers": layers,
            "outputs": outputs, "act": act, "word_bits": word_bits, "real_io": real_io}


def _train(name, frames, hidden, layers, outputs, products, inputs=440):
    return {"name": name, "kind": "train", "frames": frames, "inputs": inputs, "hidden": hidden, "layers": layers,
            "outputs": outputs, "products": products}


def listed():
    return [
        # on-device recognition, one frame every 10 ms: latency of a whole pass, 3.4 MB of packed weights
        _forward("one-frame", 1, 2048, 6, 3400, SIGN),
        # the same with the network the paper deploys (real weights at both ends), a few frames buffered
        _forward("few-frames-mixed", 16, 2048, 6, 3400, MIXED, real_io=True),
        # a small network on a short block of frames
        _forward("small-network", 64, 512, 3, 1000, SIGN),
        # one utterance (a few seconds) on the paper's 1024-unit network, 3307 tied states
        _forward("utterance", 333, 1024, 6, 3307, SIGN),
        # one utterance on the mixed topology with binary weights everywhere
        _forward("utterance-mixed", 600, 2048, 6, 3400, MIXED),
        # a block of utterances on the paper's 2048-unit network with {0, 1} units, 3972 tied states, 64-bit words
        _forward("block-step01", 1500, 2048, 6, 3972, STEP01, word_bits=64),
        # the benchmark's batch
        _forward("batch", 4096, 2048, 6, 3400, SIGN),
        # the same batch with real activations
        _forward("batch-hardtanh", 4096, 2048, 6, 3400, HARDTANH),
        # the same batch on the network the paper deploys
        _forward("batch-mixed", 4096, 2048, 6, 3400, MIXED, real_io=True),
        # offline scoring of a large batch on the widest network
        _forward("large-batch", 16384, 4096, 6, 4000, SIGN, word_bits=64),
        # training: a small minibatch with every product in ascending order
        _train("train-small", 256, 2048, 6, 3400, "ascending"),
        # training: a large minibatch, the gradient products of the binary layers on the int8 matrix cores
        _train("train-large", 4096, 2048, 6, 3400, "int8"),
    ]


def _macs(case):
    h = case["hidden"]
    return case["inputs"] * h + (case["layers"] - 1) * h * h + h * case["outputs"]


def _log_uniform(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _width(rng, lo, hi, step):
    """Mostly multiples of `step`, as networks are built; some of 32; some arbitrary."""
    v, how = _log_uniform(rng, lo, hi), rng.random()
    if how < 0.55:
        return max(lo, min(hi, round(v / step) * step))
    return max(lo, min(hi, round(v / 32) * 32)) if how < 0.85 else v


def draw(rng):
    case = {"inputs": rng.choice([440, 440, 440, 429, 360, 143, 520]), "hidden": _width(rng, 512, 4096, 512),
            "layers": rng.randint(3, 6), "outputs": _width(rng, 1000, 4000, 100)}
    if rng.random() < 0.15:
        products = rng.choice(["ascending", "int8"])
        # no dearer than the listed training steps
        most = 4096 * 28.75e6 if products == "int8" else 512 * 28.75e6
        top = max(32, min(4096, int(most / _macs(case))))
        case.update(kind="train", products=products, frames=_log_uniform(rng, 32, top))
        return case
    act = rng.choice([SIGN, SIGN, SIGN, STEP01, HARDTANH, MIXED, MIXED])
    # no dearer than the listed batches of the same family
    most = 16384 * 102.0e6 if act in (SIGN, STEP01) else 4096 * 28.75e6
    top = max(1, min(16384, int(most / _macs(case))))
    case.update(kind="forward", act=act, word_bits=rng.choice([32, 64]), real_io=act == MIXED and rng.random() < 0.5,
                frames=_log_uniform(rng, 1, top))
    return case


# ---------------------------------------------------------------------------------------------------- preparation

def _dims(case):
    return [case["inputs"]] + [case["hidden"]] * case["layers"] + [case["outputs"]]


def _hidden_acts(case):
    n = case["layers"]
    if case.get("act") == MIXED:
        return ["sigmoid"] + [SIGN] * (n - 2) + ["sigmoid"]
    return [case.get("act", SIGN)] * n


def _stream():
    return torch.cuda.current_stream().cuda_stream


def _empty(*shape, dtype=torch.float32):
    return torch.empty(shape, dtype=dtype, device=DEV)


def _words(rows, n, word_bits):
    return _empty(rows, bnn.bnn_packed_words(n, word_bits), dtype=torch.int32 if word_bits == 32 else torch.int64)


def _generator(seed):
    g = torch.Generator(device=DEV)
    g.manual_seed(int(seed))
    return g


def _uniform(g, *shape):
    # odd multiples of 2^-24 in (-1, 1): no zeros, exactly representable
    i = torch.randint(0, 1 << 24, shape, generator=g, device=DEV, dtype=torch.int32)
    return (i * 2 + 1 - (1 << 24)).to(torch.float32) * 2.0 ** -24


def _normal(g, *shape, std=1.0):
    return torch.randn(*shape, generator=g, device=DEV) * std


def _prepare_forward(case, seed):
    g, wb, M, dims = _generator(seed), case["word_bits"], case["frames"], _dims(case)
    acts = _hidden_acts(case)
    keep, descs, x_binary = [], [], 0
    for l in range(len(dims) - 1):
        K, N = dims[l], dims[l + 1]
        last = l == len(dims) - 2
        W, bias = _uniform(g, N, K), _normal(g, N, std=0.1)
        d = {"K": K, "N": N, "word_bits": wb, "x_is_binary": x_binary,
             "act": bnn.BNN_ACT_LOGSOFTMAX if last else bnn.ACT_BY_NAME[acts[l]]}
        if case["real_io"] and (l == 0 or last):
            W = W * math.sqrt(3.0 / K)
            d.update(w_is_real=1, Wp=W.data_ptr(), scale=0, bias=bias.data_ptr())
            keep += [W, bias]
        else:
            Wp, alpha = _words(N, K, wb), _empty(1)
            bnn.bnn_pack_weights(W.data_ptr(), N, K, wb, Wp.data_ptr(), alpha.data_ptr(), _stream())
            scale = alpha.expand(N).contiguous()
            d.update(Wp=Wp.data_ptr(), scale=scale.data_ptr(), bias=bias.data_ptr())
            keep += [Wp, scale, bias]
        descs.append(d)
        if not last:
            x_binary = {SIGN: 1, STEP01: 2}.get(acts[l], 0)
    layers = bnn.make_layer_array(descs)
    nbytes = bnn.bnn_forward_workspace_bytes(layers, len(descs), M)
    return {"kind": "forward", "keep": keep, "layers": layers, "n": len(descs), "M": M, "X": _normal(g, M, dims[0]),
            "out": _empty(M, dims[-1]), "ws": _empty(max(nbytes, 256), dtype=torch.uint8), "ws_bytes": nbytes}


def _prepare_train(case, seed):
    g, M, dims, wb = _generator(seed), case["frames"], _dims(case), 32
    L = len(dims) - 1
    W = [_uniform(g, dims[l + 1], dims[l]) for l in range(L)]
    s = {"kind": "train", "M": M, "dims": dims, "int8": case["products"] == "int8", "W": W,
         "r": [_normal(g, dims[l + 1], std=0.1) for l in range(L)], "X": _normal(g, M, dims[0]),
         "labels": torch.randint(0, dims[-1], (M,), generator=g, device=DEV, dtype=torch.int32)}
    s["Wp"] = [_words(dims[l + 1], dims[l], wb) for l in range(L)]
    s["WpT"] = [_words(dims[l], dims[l + 1], wb) for l in range(L)]
    s["hhat"] = [_empty(M, n) for n in dims[1:]]
    s["bits"] = [_words(M, n, wb) for n in dims[1:-1]]
    s["hT"] = [_words(n, M, wb) for n in dims[1:-1]]
    s["g"] = [_empty(M, n) for n in dims[1:]]
    s["gT"] = [_empty(n, M) for n in dims[1:]]
    s["XT"] = _empty(dims[0], M)
    s["gW"] = [_empty(dims[l + 1], dims[l]) for l in range(L)]
    s["gr"] = [_empty(n) for n in dims[1:]]
    s["norm"] = [_empty(1) for _ in range(L)]
    s["clip_ws"] = _empty(2048, dtype=torch.uint8)
    need = max([bnn.bnn_layer_binw_realx_i8_workspace_bytes(n, M, k) for k, n in zip(dims, dims[1:])] +
               [bnn.bnn_layer_binw_realx_i8_workspace_bytes(M, n, k) for k, n in zip(dims, dims[1:])])
    s["i8_bytes"], s["i8_ws"] = need, _empty(need, dtype=torch.uint8)
    # the device addresses, looked up once
    s["p"] = {k: [t.data_ptr() for t in v] for k, v in s.items() if isinstance(v, list) and isinstance(v[0], torch.Tensor)}
    return s


def prepare(case, seed):
    return _prepare_forward(case, seed) if case["kind"] == "forward" else _prepare_train(case, seed)


# ---------------------------------------------------------------------------------------------------- one pass

def _run_train(s):
    """One minibatch: binary weights and activations, cut-off k = 1, gradient norms clipped at 15, learning rate 1e-3."""
    st, p, M, dims, wb = _stream(), s["p"], s["M"], s["dims"], 32
    L = len(dims) - 1
    X, XT, labels, i8, i8_bytes = (s["X"].data_ptr(), s["XT"].data_ptr(), s["labels"].data_ptr(), s["i8_ws"].data_ptr(),
                                   s["i8_bytes"])
    for l in range(L):
        K, N = dims[l], dims[l + 1]
        bnn.bnn_pack_weights(p["W"][l], N, K, wb, p["Wp"][l], 0, st)
        if l:
            bnn.bnn_pack_weights_transposed(p["W"][l], N, K, wb, p["WpT"][l], st)
    for l in range(L):
        K, N = dims[l], dims[l + 1]
        act = bnn.BNN_ACT_LINEAR if l < L - 1 else bnn.BNN_ACT_LOGSOFTMAX
        if l == 0:
            bnn.bnn_layer_binw_realx(X, p["Wp"][0], 0, p["r"][0], M, K, N, act, wb, p["hhat"][0], st)
        else:
            bnn.bnn_layer_binw_binx(p["bits"][l - 1], p["Wp"][l], 0, p["r"][l], M, K, N, act, wb, p["hhat"][l], st)
        if l < L - 1:
            bnn.bnn_pack_activations(p["hhat"][l], M, N, wb, p["bits"][l], st)
    bnn.bnn_softmax_xent_grad(p["hhat"][L - 1], labels, M, dims[-1], p["g"][L - 1], st)
    for l in range(L - 1, -1, -1):
        K, N = dims[l], dims[l + 1]
        g, gT, gW = p["g"][l], p["gT"][l], p["gW"][l]
        if l < L - 1:
            bnn.bnn_mask_grad(g, p["hhat"][l], M * N, 1.0, g, st)
        bnn.bnn_transpose_f32(g, M, N, gT, st)
        if l == 0:
            bnn.bnn_transpose_f32(X, M, K, XT, st)
            bnn.bnn_backward_weight(gT, XT, N, K, M, gW, st)
        else:
            bnn.bnn_pack_weights_transposed(p["hhat"][l - 1], M, K, wb, p["hT"][l - 1], st)
            if s["int8"]:
                bnn.bnn_layer_binw_realx_i8(gT, p["hT"][l - 1], 0, 0, N, M, K, wb, gW, i8, i8_bytes, st)
                bnn.bnn_layer_binw_realx_i8(g, p["WpT"][l], 0, 0, M, N, K, wb, p["g"][l - 1], i8, i8_bytes, st)
            else:
                bnn.bnn_backward_weight_binh(gT, p["hT"][l - 1], N, K, M, wb, gW, st)
                bnn.bnn_backward_input_binw(g, p["WpT"][l], M, N, K, wb, p["g"][l - 1], st)
        bnn.bnn_bias_grad(g, M, N, p["gr"][l], st)
    clip_ws = s["clip_ws"].data_ptr()
    for l in range(L):
        K, N = dims[l], dims[l + 1]
        bnn.bnn_grad_norm_clip(p["gW"][l], N * K, 15.0, clip_ws, p["norm"][l], st)
        bnn.bnn_update_clip(p["W"][l], p["gW"][l], N * K, 1e-3, 1, st)
        bnn.bnn_update_clip(p["r"][l], p["gr"][l], N, 1e-3, 0, st)
    return {"logp": s["hhat"][L - 1], "W": s["W"], "r": s["r"], "gW": s["gW"], "gr": s["gr"], "norm": s["norm"]}


def run(state):
    if state["kind"] == "train":
        return _run_train(state)
    bnn.bnn_forward(state["layers"], state["n"], state["X"].data_ptr(), state["M"], state["out"].data_ptr(),
                    state["ws"].data_ptr(), state["ws_bytes"], _stream())
    return state["out"]


# ---------------------------------------------------------------------------------------------------- what a pass needs

def work(case):
    """Bytes: frames in, log-posteriors out, the model once (training: gradients and updated weights written too).
    Flops: two per weight and frame, three such products per layer in training (no input gradient at the first)."""
    M, dims = case["frames"], _dims(case)
    pairs = list(zip(dims, dims[1:]))
    macs = _macs(case)
    if case["kind"] == "train":
        params = macs + sum(dims[1:])
        return {"bytes": 4.0 * (M * dims[0] + M * dims[-1] + 3 * params + M), "flops": 2.0 * M * (3 * macs - dims[0] * dims[1])}
    weights = 0
    for l, (k, n) in enumerate(pairs):
        real = case["real_io"] and l in (0, len(pairs) - 1)
        weights += n * (4 * k + 4 if real else 4 * ((k + 31) // 32) + 8)
    return {"bytes": 4.0 * M * (dims[0] + dims[-1]) + weights, "flops": 2.0 * M * macs}


def tolerance(case):
    """fp32 log-posteriors: binary units are decided exactly, what remains is the rounding of fp32 sums and of the
    log-Softmax.  Training with int8 gradient products: sums within K 2^-27 of a row's largest gradient, about 1e-5 of a
    typical sum, passed down the layers."""
    if case["kind"] == "train" and case["products"] == "int8":
        return {"rel": 1e-4, "max": 5e-3}
    return {"rel": 1e-5, "max": 4e-4}
