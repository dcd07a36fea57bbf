"""What a program built on this library has it do, as measurable cases.

A case is one pass through the public entry points on data that is already where such a program has it: ciphertexts
of the service side on the GPU, slot vectors and images of the client side on the host.  The contexts, keys and plans
(weights converted and encoded ahead of time) are made once per parameter set and kept, as a program keeps them.

    rotate     rotLeft of a batch of ciphertexts: the key-switched operation the networks are dominated by
    hoist      several rotations of the same ciphertexts (the taps of a convolution, the corners of a pool)
    multiply   ciphertext product, relinearisation, rescale: what an activation does
    linear     plaintext product, sum, rescale: one term of a linear layer
    client     encode and encrypt slot vectors, decrypt and decode them: the two ends of every program
    network    encrypted inference of one image, from the image to the decrypted scores

Both arithmetics of the library occur: primes below 2^50 on 2^12 <= N <= 2^15 (fp64 kernels) and anything else up to
60 bits (integer kernels).
"""
import ctypes
import math

import numpy as np
import torch

from paper_1810_00845_amd import hisa, nets, synth


def _prm(log_n, limbs, bits, dnum, special_bits=50, first_bits=None, level=None):
    return {"log_n": log_n, "limbs": limbs, "level": level or limbs, "first_bits": first_bits or bits, "bits": bits,
            "dnum": dnum, "special_bits": special_bits}


def listed():
    return [
        # the smallest call: one rotation under the parameters of a single small convolution (30-bit primes, 60-bit
        # special prime: integer kernels), where launches and host work are everything
        dict(_prm(12, 3, 30, 3, special_bits=60), name="rotate_one_n12", op="rotate", batch=1, step=1),
        # one rotation under the small network's parameters: latency of a program that rotates ciphertext by ciphertext
        dict(_prm(13, 8, 40, 2, first_bits=50), name="rotate_one_n13", op="rotate", batch=1, step=7),
        # the few ciphertexts of a layer of the largest network, some levels down (last digit of the key switch ragged)
        dict(_prm(15, 21, 45, 3, first_bits=50, level=17), name="rotate_few_n15", op="rotate", batch=3, step=64),
        # throughput: the primitive micro-benchmark at its largest point
        dict(_prm(15, 16, 50, 3), name="rotate_batch_n15", op="rotate", batch=64, step=1),
        # primes beyond 50 bits (higher precision scales): the integer kernels at the same ring degree
        dict(_prm(15, 8, 58, 3, special_bits=60), name="rotate_wide_n15", op="rotate", batch=16, step=7),
        # the 24 rotated taps of a 5x5 convolution over one ciphertext, under the medium network's parameters
        dict(_prm(14, 12, 40, 3, first_bits=50), name="hoist_taps_n14", op="hoist", batch=1, steps=24),
        # activations of a wide layer: an odd number of ciphertexts at an odd level
        dict(_prm(14, 16, 50, 3, level=11), name="multiply_n14", op="multiply", batch=37),
        # a masked / weighted sum of ciphertexts
        dict(_prm(14, 8, 50, 1), name="linear_n14", op="linear", batch=24),
        # a client's vectors, complex-free and full length
        dict(_prm(14, 12, 40, 3, first_bits=50), name="client_n14", op="client", batch=4),
        # the three benchmark networks in the layout that the cost model picks for them
        {"name": "lenet_small", "op": "network", "net": "lenet_small", "layout": "chw_fc"},
        {"name": "lenet_medium", "op": "network", "net": "lenet_medium", "layout": "chw_fc"},
        {"name": "squeezenet_cifar", "op": "network", "net": "squeezenet_cifar", "layout": "chw"},
    ]


def _log_int(rng, lo, hi):
    return min(hi, int(math.exp(rng.uniform(math.log(lo), math.log(hi + 1)))))


def draw(rng):
    op = rng.choice(["rotate", "rotate", "rotate", "wide", "hoist", "multiply", "multiply", "linear", "client", "network"])
    if op == "network":      # the small network's sequence of layers over other images, filters and widths
        side, filt = rng.randrange(14, 31), rng.choice([3, 5])
        return {"op": "network", "net": "generic", "layout": rng.choice(["hw", "chw_fc"]), "log_n": rng.choice([13, 14]),
                "side": side, "filt": filt, "stride": 2, "channels": rng.randrange(2, 9), "hidden": _log_int(rng, 8, 100),
                "classes": rng.randrange(2, 12)}
    if op == "wide":
        limbs = rng.randrange(2, 9)
        return dict(_prm(rng.randrange(11, 17), limbs, rng.randrange(51, 59), min(limbs, rng.randrange(1, 4)), special_bits=60,
                         level=rng.randrange(2, limbs + 1)), op="rotate", batch=_log_int(rng, 1, 16), step=rng.randrange(1, 512))
    log_n, limbs = rng.randrange(12, 16), rng.randrange(2, 22)
    prm = _prm(log_n, limbs, rng.randrange(38, 51), min(limbs, rng.randrange(1, 4)), first_bits=50, level=rng.randrange(2, limbs + 1))
    if op == "hoist":
        return dict(prm, op=op, batch=_log_int(rng, 1, 4), steps=rng.randrange(2, 25))
    if op == "client":
        return dict(prm, op=op, batch=_log_int(rng, 1, 8))
    if op == "rotate":
        return dict(prm, op=op, batch=_log_int(rng, 1, 64), step=rng.randrange(1, 1024))
    return dict(prm, op=op, batch=_log_int(rng, 1, 64))


# --- what a program keeps: one context with its keys, and the plans of one network ---

_kept = {}


def _keep(key, make):
    if key not in _kept:
        _kept.clear()        # one parameter set at a time: the keys and plans of another case are given back
        _kept[key] = make()
    return _kept[key]


def _context(case):
    steps = (case["step"],) if case["op"] == "rotate" else tuple(range(1, case["steps"] + 1)) if case["op"] == "hoist" else ()
    relin = case["op"] == "multiply"

    def make():
        ctx = hisa.Context(case["log_n"], [case["first_bits"]] + [case["bits"]] * (case["limbs"] - 1), case["dnum"],
                           case["special_bits"], seed=1)
        if relin:
            ctx.keygen()
        ctx.gen_rot_keys(steps)
        return ctx
    return _keep(("context", relin, steps) + tuple(case[k] for k in ("log_n", "limbs", "first_bits", "bits", "dnum", "special_bits")), make)


def _network(case):
    """(parameters, layers, image of the seed) of a network case."""
    if case["net"] != "generic":
        params, layers, x = getattr(nets, case["net"])()
        side = 28 if case["net"].startswith("lenet") else x.shape[2]
        return params, layers, x.shape, side
    f, c, side = case["filt"], case["channels"], case["side"]
    out = (side - f) // case["stride"] + 1
    layers = [("conv", synth.conv_weights(3, f, f, 1, c, dist="normal", std=1.0 / f), case["stride"]),
              ("act", 1.0, 0.0),
              ("fc", synth.fc_weights(4, case["hidden"], c, out, out, std=1.0 / math.sqrt(c * out * out))),
              ("act", 1.0, 0.0),
              ("fc", synth.fc_weights(5, case["classes"], case["hidden"], 1, 1, std=1.0 / math.sqrt(case["hidden"])))]
    params = dict(log_n=case["log_n"], q_bits=[50] + [40] * 7, dnum=2, special_bits=50, scale=2.0 ** 40)
    return params, layers, (1, 1, side, side), side


class _Server:
    """A network's context, keys and plans."""

    def __init__(self, case):
        self.params, self.layers, self.shape, self.side = _network(case)
        p = self.params
        self.ctx = hisa.Context(p["log_n"], p["q_bits"], p["dnum"], p["special_bits"], seed=11)
        self.ctx.keygen()
        self.plans = {}
        self.options = dict(border=p.get("border", 0), plans=self.plans, layout=case["layout"], layer_times=False)
        self.infer(self.image(0), make_keys=True)

    def __del__(self):
        try:
            nets.free_plans(self.ctx, self.plans)
        except Exception:
            pass

    def image(self, seed):
        x = np.zeros(self.shape)
        edge = (self.shape[2] - self.side) // 2      # a zero border where the network's image has one
        x[0, :, edge:edge + self.side, edge:edge + self.side] = synth.image(seed, self.shape[1], self.side, self.side)
        return x

    def infer(self, x, **kw):
        return nets.run_encrypted(self.ctx, self.layers, x, self.params["scale"], len(self.params["q_bits"]), **self.options, **kw)[0]


def prepare(case, seed):
    if case["op"] == "network":
        server = _keep(("network",) + tuple(sorted((k, v) for k, v in case.items() if k != "name")), lambda: _Server(case))
        return {"op": "network", "server": server, "image": server.image(seed)}
    ctx = _context(case)
    n, level = case["batch"], case["level"]
    state = {"op": case["op"], "ctx": ctx}
    if case["op"] == "client":
        rng = np.random.default_rng(seed)
        return dict(state, vectors=list(rng.uniform(-1.0, 1.0, (n, ctx.slots))), scale=2.0 ** 40 if level > 1 else 2.0 ** 30, level=level)
    scale = 2.0 ** 40
    state["a"] = ctx.ct_random_batch(n, level, scale, 1000003 * seed)      # uniform residues: what encryptions look like
    if case["op"] == "rotate":
        state["step"] = case["step"]
    elif case["op"] == "hoist":
        state["steps"] = list(range(1, case["steps"] + 1))
    else:
        state["b"] = ctx.ct_random_batch(n, level, scale, 1000003 * seed + 500000)
        if case["op"] == "linear":
            slots = np.random.default_rng(seed).uniform(-1.0, 1.0, ctx.slots)
            state["w"] = ctx.encode(slots, float(ctx.primes[level - 1]), level)
            state["b"] = ctx.mul_plain_batch(state["b"], state["w"])       # the running sum: products of earlier terms
    return state


class _OnDevice:
    """The residues of neighbouring ciphertext handles as an array on the GPU; keeps the handles alive."""

    def __init__(self, cts):
        self.cts = cts
        limbs, polys, _ = cts[0].info()
        ptr = ctypes.c_uint64()
        first = None
        for ct in (cts[0], cts[-1]):
            ct.ctx._ck(hisa.load().hisa_ct_device_ptr(ctypes.c_void_p(ct.h), ctypes.byref(ptr)))
            first = ptr.value if first is None else first
        assert ptr.value - first == (len(cts) - 1) * polys * limbs * cts[0].ctx.N * 8, "not one allocation"
        self.__cuda_array_interface__ = {"shape": (len(cts), polys, limbs, cts[0].ctx.N), "typestr": "<i8", "version": 2,
                                         "data": (first, False), "strides": None}


def _residues(cts):
    return torch.as_tensor(_OnDevice(cts), device="cuda")


def run(state):
    op = state["op"]
    if op == "network":
        return state["server"].infer(state["image"])
    ctx = state["ctx"]
    if op == "client":
        cts = ctx.encrypt_batch([ctx.encode(v, state["scale"], state["level"]) for v in state["vectors"]])
        return [ctx.decode(ctx.decrypt(ct)) for ct in cts]
    a = state["a"]
    if op == "rotate":
        return _residues(ctx.rot_left_batch(a, state["step"]) if len(a) > 1 else [ctx.rot_left(a[0], state["step"])])
    if op == "hoist":
        return [_residues(row) for row in ctx.rot_left_hoisted_batch(a, state["steps"])]
    if op == "multiply":
        out = ctx.mul_no_relin_batch(a, state["b"])
        ctx.relinearize_batch(out)
    else:
        out = ctx.add_batch(ctx.mul_plain_batch(a, state["w"]), state["b"])
    ctx.rescale_batch(out)
    return _residues(out)


# --- what a pass cannot do without ---

def _transform_ops(log_n):
    """Operations of one transform: a butterfly is a modular product (8), a sum and a difference."""
    return 10.0 * (1 << (log_n - 1)) * log_n


def _key_switch(log_n, level, limbs, dnum):
    """(bytes of the key at this level, operations before the inner product, of it, after it) of one key switch."""
    n = float(1 << log_n)
    alpha = -(-limbs // dnum)
    sizes = [min(alpha, level - lo) for lo in range(0, level, alpha)]
    ext = level + alpha
    up = level * _transform_ops(log_n) + sum((ext - s) * (_transform_ops(log_n) + 9 * s * n) for s in sizes)
    inner = 18.0 * len(sizes) * ext * n
    down = (2 * alpha + 2 * level) * _transform_ops(log_n) + 2 * level * 9 * alpha * n
    return len(sizes) * 2 * ext * 8 * n, up, inner, down


def work(case):
    if case["op"] == "network":
        params, layers, shape, _ = _network(case)
        log_n, n, level = params["log_n"], float(1 << params["log_n"]), len(params["q_bits"])
        total_bytes, ops = 8.0 * shape[1] * shape[2] * shape[3] + 8.0 * 10, 0.0
        for layer in layers:         # one relinearisation per activation; a linear layer's weights and one division by P
            key, up, inner, down = _key_switch(log_n, level, len(params["q_bits"]), params["dnum"])
            ops += up + inner + down
            weights = [w for w in layer[1:] if isinstance(w, np.ndarray)]
            total_bytes += key + sum(8.0 * w.size for w in weights)
            ops += sum(2.0 * w.size * level * 18 for w in weights)
            level = max(2, level - 1)
        return {"bytes": total_bytes, "flops": ops}
    log_n, n, level, batch = case["log_n"], float(1 << case["log_n"]), case["level"], case["batch"]
    ct = 2.0 * level * 8 * n
    key, up, inner, down = _key_switch(log_n, level, case["limbs"], case["dnum"])
    rescale = (2 * level) * _transform_ops(log_n)
    if case["op"] == "rotate":
        return {"bytes": 2 * ct * batch + key, "flops": batch * (up + inner + down)}
    if case["op"] == "hoist":
        return {"bytes": ct * batch + case["steps"] * (key + ct * batch), "flops": batch * (up + case["steps"] * (inner + down))}
    if case["op"] == "multiply":
        return {"bytes": batch * (2 * ct + ct * (level - 1) / level) + key,
                "flops": batch * (4 * 9 * level * n + up + inner + down + rescale)}
    if case["op"] == "linear":
        return {"bytes": batch * (2 * ct + ct * (level - 1) / level) + ct / 2, "flops": batch * (2 * 9 * level * n + rescale)}
    # client: two transforms over the slots, the limbs' transforms of message, error and mask, and of the decryption
    fft = 10.0 * (n / 4) * (log_n - 1)
    return {"bytes": batch * (8.0 * n / 2 + 16.0 * n / 2), "flops": batch * (2 * fft + 4 * level * _transform_ops(log_n) + 2 * 8 * level * n)}


def tolerance(case):
    # Ciphertexts are whole numbers.  What a client decodes carries fresh encryption noise each time: 3.2 sqrt(N) / scale
    # per slot, 1e-9 of the values at most; the networks' scores carry that of every key switch and rescale on the way.
    if case["op"] == "network":
        return {"rel": 2e-6, "max": 2e-5}
    if case["op"] == "client":
        return {"rel": 1e-8, "max": 1e-7}
    return "exact"
