"""The engine's work as its users meet it, for timing and for comparing outputs.

A case is one pass of a part of Algorithm 1 (or of the late joiner's catch-up
and the 4-bit variant) through the public calls of
``paper_2306_10015_amd.mezo``, on parameter sets of the shapes in
``synth.WORKLOADS`` and on generic ones:

  sample    the inner loop over a machine's samples: +eps, -2 eps, and the
            restore fused with the next sample's +eps: one or two records a
            sweep
  update    the apply loop of one iteration over K one-byte gradients
  restore   the same out of place, from the weights' backup
  replay    a late joiner's catch-up over T logged iterations of K gradients
  checksum  ChecksumMatch: the 64-bit checksum of every weight
  convert   dense weights to 4-bit storage and back, tensor by tensor, what a
            forward pass over 4-bit weights needs

``set`` is a workload's name, or ``opt:d,ffn,layers,vocab`` (the decoder shapes
of ``synth``) or ``mats:n,rows,cols`` (n equal matrices).
"""
from __future__ import annotations

import math

import numpy as np
import torch

from paper_2306_10015_amd import mezo, synth

EPS = 1e-3
#: Per-gradient learning rate: at weights of 0.02 an update of K gradients
#: moves most of them by a storage step or more, so that a wrong one shows.
LR = 1e-4
#: Alignment of each tensor within its set's buffer, in bytes.
ALIGN = 256


def listed():
    return [
        # the smallest set: one sample's three sweeps, all launch and latency
        {"name": "sample_tiny_f32", "op": "sample", "set": "tiny", "storage": "f32", "gaussian": "fast",
         "samples": 1, "K": 0, "T": 0, "codec": "linear"},
        # one sample on a small model in full precision: sweeps bound by memory
        {"name": "sample_opt125m_f32", "op": "sample", "set": "opt125m", "storage": "f32", "gaussian": "fast",
         "samples": 1, "K": 0, "T": 0, "codec": "linear"},
        # a machine's loop over samples on a mid-size model in bf16
        {"name": "samples4_opt1.3b_bf16", "op": "sample", "set": "opt1.3b", "storage": "bf16", "gaussian": "fast",
         "samples": 4, "K": 0, "T": 0, "codec": "linear"},
        # one iteration's apply loop, few gradients, full precision, noise every device reproduces
        {"name": "update_opt125m_f32_k8_portable", "op": "update", "set": "opt125m", "storage": "f32",
         "gaussian": "portable", "samples": 0, "K": 8, "T": 0, "codec": "linear"},
        # the ordinary apply loop: four machines with four samples each
        {"name": "update_opt1.3b_bf16_k16", "op": "update", "set": "opt1.3b", "storage": "bf16", "gaussian": "fast",
         "samples": 0, "K": 16, "T": 0, "codec": "linear"},
        # the paper's model size with 64 gradients: the largest pass
        {"name": "update_opt6.7b_bf16_k64", "op": "update", "set": "opt6.7b", "storage": "bf16", "gaussian": "fast",
         "samples": 0, "K": 64, "T": 0, "codec": "linear"},
        # restore from the backup and apply, on tensors of odd sizes, signed-log gradients
        {"name": "restore_ragged_bf16_k5", "op": "restore", "set": "opt:701,2803,6,9973", "storage": "bf16",
         "gaussian": "fast", "samples": 0, "K": 5, "T": 0, "codec": "log"},
        # a late joiner that missed six iterations of a small model
        {"name": "replay_opt125m_f32_6x8", "op": "replay", "set": "opt125m", "storage": "f32", "gaussian": "fast",
         "samples": 0, "K": 8, "T": 6, "codec": "linear"},
        # a machine's samples on 4-bit weights
        {"name": "samples2_opt1.3b_nf4", "op": "sample", "set": "opt1.3b", "storage": "nf4", "gaussian": "fast",
         "samples": 2, "K": 0, "T": 0, "codec": "linear"},
        # the apply loop on 4-bit weights
        {"name": "update_opt1.3b_nf4_k16", "op": "update", "set": "opt1.3b", "storage": "nf4", "gaussian": "fast",
         "samples": 0, "K": 16, "T": 0, "codec": "linear"},
        # an embedding to 4-bit storage and back to bf16
        {"name": "convert_embedding_bf16", "op": "convert", "set": "mats:1,50272,2048", "storage": "bf16",
         "gaussian": "fast", "samples": 0, "K": 0, "T": 0, "codec": "linear"},
        # replicas compare their weights after an iteration
        {"name": "checksum_opt125m_f32", "op": "checksum", "set": "opt125m", "storage": "f32", "gaussian": "fast",
         "samples": 0, "K": 0, "T": 0, "codec": "linear"},
    ]


def draw(rng):
    """One more case: every path, storage type, option and set shape above,
    sizes over their logarithm from the smallest set's to the 1.3B model's."""
    op = rng.choice(["sample", "sample", "update", "update", "restore", "replay", "checksum", "convert"])
    storage = rng.choice(["f32", "bf16"] if op == "convert" else ["f32", "bf16", "bf16", "nf4"])
    gaussian = "portable" if op not in ("checksum", "convert") and rng.random() < 0.25 else "fast"
    K = T = samples = 0
    if op == "sample":
        samples = rng.randint(1, 4)
    if op in ("update", "restore"):
        K = int(round(math.exp(rng.uniform(0.0, math.log(64.0)))))
    if op == "replay":
        T, K = rng.randint(2, 8), rng.randint(1, 32)
    records = max(1, 3 * samples, K * max(1, T))
    # at most 2^30 elements and 2^33.5 elements x records (a pass of a few ms)
    top = min(30.0, 33.5 - math.log2(records))
    target = 2.0 ** rng.uniform(20.0 if op != "convert" else 18.0, top)
    if rng.random() < 0.3:
        n = rng.randint(1, 24)
        rows = max(1, int(round(math.sqrt(target / n))))
        spec = f"mats:{n},{rows},{max(1, int(round(target / n / rows)))}"
    else:
        layers = rng.randint(1, 24)
        # target = 12 layers d^2 + 8 d^2 (a vocabulary of 8 d)
        d = max(16, int(round(math.sqrt(target / (12 * layers + 8)))))
        if rng.random() < 0.7:
            d = max(16, d // 8 * 8)
        spec = f"opt:{d},{4 * d + rng.choice([0, 0, 1])},{layers},{8 * d + rng.randint(0, 7)}"
    return {"op": op, "set": spec, "storage": storage, "gaussian": gaussian, "samples": samples, "K": K, "T": T,
            "codec": rng.choice(["linear", "linear", "log"]) if K else "linear"}


# ---- the parameter sets -------------------------------------------------------

def _sizes(spec):
    """Elements of every tensor of a set, in registration order (= tensor_id)."""
    kind, _, rest = spec.partition(":")
    if kind in synth.WORKLOADS:
        return [int(math.prod(s)) for _, s in synth.WORKLOADS[kind].shapes]
    v = [int(x) for x in rest.split(",")]
    if kind == "mats":
        n, rows, cols = v
        return [rows * cols] * n
    d, ffn, layers, vocab = v
    layer = [d * d] * 4 + [d * ffn] * 2 + [d] * 4
    return [vocab * d] + layer * layers + [d, d]


def _layout(sizes, per_align):
    """Start of every tensor in one buffer (multiples of per_align), and its length."""
    starts, total = [], 0
    for n in sizes:
        starts.append(total)
        total += (n + per_align - 1) // per_align * per_align
    return starts, total


def _dense(sizes, dtype, seed):
    """Weights N(0, 0.02) in one buffer (zero between the tensors)."""
    g = torch.Generator(device="cuda")
    g.manual_seed(seed)
    starts, total = _layout(sizes, ALIGN // dtype.itemsize)
    flat = torch.zeros(total, dtype=dtype, device="cuda")
    for s, n in zip(starts, sizes):
        flat[s:s + n].copy_(torch.empty(n, dtype=torch.float32, device="cuda").normal_(0.0, 0.02, generator=g))
    return flat, [flat[s:s + n] for s, n in zip(starts, sizes)]


def _nf4(sizes, seed):
    """4-bit weights: uniform codes (NF4's values are normal quantiles) and the
    absmax that blocks of 64 weights N(0, 0.02) have; zeros without a seed."""
    g = torch.Generator(device="cuda")
    g.manual_seed(seed or 0)
    cs, ctotal = _layout([(n + 1) // 2 for n in sizes], ALIGN)
    bs, btotal = _layout([(n + 63) // 64 for n in sizes], ALIGN // 4)
    codes = torch.zeros(ctotal, dtype=torch.uint8, device="cuda")
    absmax = torch.zeros(btotal, dtype=torch.float32, device="cuda")
    views = []
    for c, b, n in zip(cs, bs, sizes):
        cv, bv = codes[c:c + (n + 1) // 2], absmax[b:b + (n + 63) // 64]
        if seed is not None:
            cv.random_(0, 256, generator=g)
            if n % 2:
                cv[-1] &= 15
            bv.uniform_(0.04, 0.06, generator=g)
        views.append(mezo.NF4Tensor(cv, bv, n))
    return codes, absmax, views


_DTYPES = {"f32": torch.float32, "bf16": torch.bfloat16}


def _records(case, seed):
    """Seeds and one-byte gradients of every step: (machine, step, sample)
    ascending, machines by their 64-bit identifiers."""
    rng = np.random.default_rng([int(seed), 77])
    steps = []
    first = int(rng.integers(0, 100_000))
    # the four (or more) machines of the run and how many samples each sends
    K = case["K"] if case["K"] else 1
    machines = np.sort(rng.integers(0, 2 ** 63, size=max(1, (K + 3) // 4), dtype=np.int64)).astype(np.uint64)
    for t in range(max(1, case["T"])):
        s = np.zeros(K, dtype=mezo.SEED_DTYPE)
        for k in range(K):
            s[k] = (machines[k // 4], first + t, k % 4)
        q = rng.integers(1, 128, size=K) * rng.choice([-1, 1], size=K)
        if case["codec"] == "log":  # codes of gradients up to about 1
            q = np.sign(q) * (1 + np.abs(q) % 64)
        steps.append((s, q.astype(np.int8)))
    return steps


def _codec(case):
    if case["codec"] == "log":
        return mezo.codec(mezo.SIGNED_LOG, alpha=64.0)
    return mezo.DEFAULT_CODEC


def _sample_seeds(case, seed):
    rng = np.random.default_rng([int(seed), 78])
    machine, step = int(rng.integers(0, 2 ** 63)), int(rng.integers(0, 100_000))
    return [(machine, step, j) for j in range(case["samples"])]


def prepare(case, seed):
    """Registered weights, and the seeds and gradients of the pass."""
    sizes = _sizes(case["set"])
    st = {"case": case, "op": case["op"]}
    if case["op"] == "convert":
        flat, views = _dense(sizes, _DTYPES[case["storage"]], seed)
        codes, absmax, nf4 = _nf4(sizes, None)
        back = torch.zeros_like(flat)
        starts, _ = _layout(sizes, ALIGN // flat.dtype.itemsize)
        st["pairs"] = [(v, t, back[s:s + n]) for v, t, s, n in zip(views, nf4, starts, sizes)]
        st["buffers"] = {"codes": codes, "absmax": absmax, "values": back}
        return st
    gauss = mezo.GAUSS_PORTABLE if case["gaussian"] == "portable" else mezo.GAUSS_FAST

    def weights(s):
        if case["storage"] == "nf4":
            codes, absmax, views = _nf4(sizes, s)
            return mezo.ParamSet(views, gaussian=gauss), {"codes": codes, "absmax": absmax}
        flat, views = _dense(sizes, _DTYPES[case["storage"]], s)
        return mezo.ParamSet(views, gaussian=gauss), {"theta": flat}

    st["ps"], st["buffers"] = weights(seed)
    if case["op"] == "restore":  # the backup: the iteration's starting weights
        st["backup"], st["backup_buffers"] = weights(seed + 1_000_003)
    if case["op"] == "checksum":
        st["sum"] = torch.zeros(1, dtype=torch.int64, device="cuda")
    st["samples"] = _sample_seeds(case, seed)
    st["steps"] = _records(case, seed)
    st["codec"] = _codec(case)
    return st


def run(st):
    """One pass."""
    op = st["op"]
    if op == "convert":
        for x, t, y in st["pairs"]:
            mezo.nf4_quantize(x, out=t)
            mezo.nf4_dequantize(t, out=y)
        return st["buffers"]
    ps = st["ps"]
    if op == "checksum":
        ps.checksum_into(st["sum"])
        return st["sum"]
    if op == "sample":
        s = st["samples"]
        ps.perturb(s[0], EPS)
        for j in range(len(s)):
            # (the forward pass for l+)
            ps.perturb(s[j], -2 * EPS)
            # (the forward pass for l-)
            if j + 1 < len(s):
                ps.perturb_multi([s[j], s[j + 1]], [EPS, EPS])
        ps.perturb(s[-1], EPS)
    elif op == "update":
        seeds, q = st["steps"][0]
        ps.update_multi(seeds, q, LR, st["codec"])
    elif op == "restore":
        seeds, q = st["steps"][0]
        ps.update_multi_from(st["backup"], seeds, q, LR, st["codec"])
    else:
        ps.replay([(seeds, q, LR) for seeds, q in st["steps"]], st["codec"])
    return st["buffers"]


# ---- what a pass cannot do without -----------------------------------------------

def _passes(case):
    """(records, storage rounds) of every sweep over the weights in one pass."""
    if case["op"] == "sample":
        n = case["samples"]
        return [1] + [1] * n + [2] * (n - 1) + [1]
    return [max(1, case["K"]) * max(1, case["T"])]


#: Operations per element and record: a counter-based generator's four words and
#: the Box-Muller transform of a block of 4 Gaussians, the weighted sum included,
#: take 62 (10 rounds of two products and two three-way xors, less what is shared).
OPS = 15.5


def work(case):
    n = sum(_sizes(case["set"]))
    stored = {"f32": 4.0, "bf16": 2.0, "nf4": 0.5 + 4.0 / 64}[case["storage"]]
    if case["op"] == "checksum":
        return {"bytes": n * stored, "flops": n * stored}
    if case["op"] == "convert":
        # dense read and codes written, codes read and dense written
        return {"bytes": 2 * n * (stored + 0.5 + 4.0 / 64), "flops": n * 8.0}
    p = _passes(case)
    return {"bytes": 2 * n * stored * len(p), "flops": OPS * n * sum(p)}


def tolerance(case):
    """About four times what the hardware-transcendental noise, the portable
    noise and the 64-bit sums were seen to differ by on the listed cases and on
    drawn ones."""
    if case["op"] in ("checksum", "convert") or case["gaussian"] == "portable":
        return "exact"  # whole numbers, or arithmetic that the definition fixes to the bit
    several = case["op"] in ("sample", "replay")  # storage rounded more than once: a flipped rounding stays
    if case["storage"] == "nf4":
        # one code flipped in an earlier step can move its block's absmax by a tenth
        blocks = max(1.0, sum(_sizes(case["set"])) / 64.0)
        if several:
            return {"rel": min(0.03, 1.2e-4 + 0.1 / math.sqrt(blocks)), "max": 0.2, "differ": 1e-5}
        return {"rel": 2e-7, "max": 2e-6, "differ": 1e-5}
    if case["storage"] == "bf16":
        return {"rel": 7e-5, "max": 0.09} if several else {"rel": 1.4e-5, "max": 0.03}
    return {"rel": 6e-7, "max": 6e-6}


# ---- the same in 64 bits, in plain torch -------------------------------------------

_M32 = 0xFFFFFFFF


def _gaussians(seed, tensor_id, block, blocks):
    """z of elements 4 block .. 4 (block + blocks) - 1 of a tensor: Philox4x32-10
    (Salmon et al., SC'11) on counter (e / 4, tensor, sample, step) and the
    machine's 64 bits as key, then Box-Muller on 24-bit uniforms."""
    machine, step, sample = (int(x) for x in seed)
    dev = "cuda"
    c0 = torch.arange(block, block + blocks, dtype=torch.int64, device=dev)
    c1, c2, c3 = (torch.full_like(c0, int(x)) for x in (tensor_id, sample, step))
    k0, k1 = machine & _M32, machine >> 32 & _M32
    for _ in range(10):
        pa, pb = c0 * 0xD2511F53, c2 * 0xCD9E8D57
        c0, c1, c2, c3 = ((pb >> 32 & _M32) ^ c1 ^ k0, pb & _M32, (pa >> 32 & _M32) ^ c3 ^ k1, pa & _M32)
        k0, k1 = (k0 + 0x9E3779B9) & _M32, (k1 + 0xBB67AE85) & _M32
    z = torch.empty(blocks, 4, dtype=torch.float64, device=dev)
    for i, (a, b) in enumerate(((c0, c1), (c2, c3))):
        r = (((a >> 8) + 1).double() * 2.0 ** -24).log_().mul_(-2.0).sqrt_()
        t = (b >> 8).double() * (2.0 ** -24 * 2.0 * math.pi)
        z[:, 2 * i] = r * t.cos()
        z[:, 2 * i + 1] = r * t.sin()
    return z.view(-1)


#: QLoRA's sixteen NF4 values in binary32.
_NF4 = [float.fromhex(h) for h in (
    "-0x1.0p+0", "-0x1.647362p-1", "-0x1.0cd65cp-1", "-0x1.94653cp-2", "-0x1.234496p-2", "-0x1.7a6a7ap-3",
    "-0x1.74f0d2p-4", "0x0p+0", "0x1.45f602p-4", "0x1.4995bep-3", "0x1.f809b4p-3", "0x1.5a066cp-2",
    "0x1.c3496ap-2", "0x1.200f52p-1", "0x1.722760p-1", "0x1.0p+0")]


def _nf4_encode(w):
    """(codes, absmax) of one tensor's values in blocks of 64."""
    n = w.numel()
    v = torch.tensor(_NF4, dtype=torch.float64, device=w.device)
    mid = ((v[1:] + v[:-1]) / 2).float().double()
    pad = torch.zeros((n + 63) // 64 * 64, dtype=torch.float64, device=w.device)
    pad[:n] = w
    a = pad.view(-1, 64).abs().amax(dim=1)
    x = pad.view(-1, 64) / torch.where(a > 0, a, torch.ones_like(a))[:, None]
    return torch.bucketize(x.view(-1)[:n].contiguous(), mid), a


def _nf4_decode(codes, a):
    v = torch.tensor(_NF4, dtype=torch.float64, device=codes.device)
    return v[codes] * a.repeat_interleave(64)[: codes.numel()]


def _pack(codes):
    c = torch.zeros((codes.numel() + 1) // 2 * 2, dtype=torch.int64, device=codes.device)
    c[: codes.numel()] = codes
    return (c[0::2] | c[1::2] << 4).to(torch.uint8)


def _coef(q, case):
    if case["codec"] == "log":
        alpha = float(np.float32(64.0))
        return -LR * math.copysign(math.expm1(abs(int(q)) / alpha), int(q))
    return -LR * int(q) * float(np.float32(1.0 / 127.0))


def _program(case, seed):
    """The steps of the pass: lists of (seed, coefficient), storage rounded after each."""
    if case["op"] == "sample":
        s, out = _sample_seeds(case, seed), []
        for x in s:
            out += [[(x, EPS)], [(x, -2 * EPS)], [(x, EPS)]]
        return out
    return [[(x, _coef(g, case)) for x, g in zip(s, q)] for s, q in _records(case, seed)]


def exact(case, seed):
    if case["op"] == "checksum":
        return None
    st = prepare(case, seed)
    sizes = _sizes(case["set"])
    cs, ctotal = _layout([(n + 1) // 2 for n in sizes], ALIGN)
    bs, btotal = _layout([(n + 63) // 64 for n in sizes], ALIGN // 4)
    if case["op"] == "convert":
        dtype = _DTYPES[case["storage"]]
        starts, total = _layout(sizes, ALIGN // dtype.itemsize)
        codes = torch.zeros(ctotal, dtype=torch.uint8, device="cuda")
        absmax = torch.zeros(btotal, dtype=torch.float64, device="cuda")
        values = torch.zeros(total, dtype=torch.float64, device="cuda")
        for i, (x, _, _) in enumerate(st["pairs"]):
            c, a = _nf4_encode(x.double())
            codes[cs[i]: cs[i] + (x.numel() + 1) // 2] = _pack(c)
            absmax[bs[i]: bs[i] + a.numel()] = a
            values[starts[i]: starts[i] + x.numel()] = _nf4_decode(c, a).to(dtype).double()
        return {"codes": codes, "absmax": absmax, "values": values}
    if sum(sizes) * sum(_passes(case)) > 2.5e10:
        return None  # (over 20 seconds in 64 bits)
    program = _program(case, seed)
    src = st["backup_buffers"] if case["op"] == "restore" else st["buffers"]
    chunk = 1 << 24  # elements at a time, a multiple of 64

    def noise(steps, tensor_id, e, n, w, rounded):
        blocks = (n + 3) // 4
        for step in steps:
            acc = torch.zeros(n, dtype=torch.float64, device="cuda")
            for s, c in step:
                acc += c * _gaussians(s, tensor_id, e // 4, blocks)[:n]
            w = rounded(w + acc)
        return w

    if case["storage"] == "nf4":
        codes = torch.zeros(ctotal, dtype=torch.uint8, device="cuda")
        absmax = torch.zeros(btotal, dtype=torch.float64, device="cuda")
        for i, n in enumerate(sizes):
            for e in range(0, n, chunk):
                m = min(chunk, n - e)
                b = src["codes"][cs[i] + e // 2: cs[i] + (e + m + 1) // 2].long()
                c = torch.stack((b & 15, b >> 4), dim=1).view(-1)[:m]
                a = src["absmax"][bs[i] + e // 64: bs[i] + (e + m + 63) // 64].double()
                held = {}

                def rounded(w):
                    held["c"], held["a"] = _nf4_encode(w)
                    return _nf4_decode(held["c"], held["a"].float().double())

                noise(program, i, e, m, _nf4_decode(c, a), rounded)
                p = _pack(held["c"])
                codes[cs[i] + e // 2: cs[i] + e // 2 + p.numel()] = p
                absmax[bs[i] + e // 64: bs[i] + e // 64 + held["a"].numel()] = held["a"]
        return {"codes": codes, "absmax": absmax}
    dtype = _DTYPES[case["storage"]]
    starts, total = _layout(sizes, ALIGN // dtype.itemsize)
    theta = torch.zeros(total, dtype=torch.float64, device="cuda")
    for i, n in enumerate(sizes):
        for e in range(0, n, chunk):
            m = min(chunk, n - e)
            w = src["theta"][starts[i] + e: starts[i] + e + m].double()
            theta[starts[i] + e: starts[i] + e + m] = noise(program, i, e, m, w, lambda x: x.to(dtype).double())
    return {"theta": theta}
