"""The work that is timed: what a program that serves a GlowQ model has the library do.

Serving calls the group and block forward (one token, a batch of decoding sequences, short
and long prompts, with and without the correction), in W4A16 and in the microscaling
variant; getting a model ready calls quantiser, weight preparation, factorisation and
importance scores.  Shapes are those of the repository's workloads (decoder layers of 7B,
8B and 13B size) and ragged relatives of them.  Operands are drawn in storage form on the
GPU: uniform nibbles, scales as round-to-nearest produces them for N(0, 0.02^2) weights,
factors of balanced magnitude, activations with per-channel spread and 1 % outlier channels.
"""
from __future__ import annotations

import math

import torch

import paper_2603_25385_amd as G

ACT = {"f16": (G.GLOWQ_F16, torch.float16), "bf16": (G.GLOWQ_BF16, torch.bfloat16),
       "f32": (G.GLOWQ_F32, torch.float32)}
STEP = 0.0073                       # (max - min) / 15 of 128 samples of N(0, 0.02^2)


# ---- cases ------------------------------------------------------------------------------
def group(d_in, d_outs, T, r, G=128, act="f16", out="act", restore=True, kind="group"):
    """One input-sharing group (or solo module): a single glowq_group_forward."""
    return {"kind": kind, "d_in": d_in, "d_outs": ",".join(map(str, d_outs)), "T": T, "r": r, "G": G,
            "act": act, "out": out, "restore": restore}


def block(hidden, kv, inter, layers, T, r, G=128, act="f16", restored=1.0):
    """`layers` decoder layers (q/k/v, o, gate/up, down) in one glowq_block_forward, a share
    of the units restored."""
    return {"kind": "block", "hidden": hidden, "kv": kv, "inter": inter, "layers": layers, "T": T, "r": r,
            "G": G, "act": act, "out": "act", "restored": restored}


def offline(d_in, d_outs, r, p, q, act="f16"):
    """Getting one unit ready: quantise, prepare, factorise, score."""
    return {"kind": "offline", "d_in": d_in, "d_outs": ",".join(map(str, d_outs)), "r": r, "p": p, "q": q,
            "G": 128, "act": act}


def listed():
    return [
        # the smallest group there is use for: what a call costs
        dict(group(256, [256] * 3, 16, 16, G=64, out="f32"), name="tiny_group_T16"),
        # one sequence decoding, one layer's q/k/v at a time
        dict(group(4096, [4096] * 3, 1, 64), name="qkv_T1"),
        # eight sequences decoding in bfloat16, gate/up of an 8B-sized layer
        dict(group(4096, [14336] * 2, 8, 128, act="bf16"), name="gateup_T8_bf16"),
        # twenty-four sequences decoding, a whole 8B-sized layer
        dict(block(4096, 1024, 14336, 1, 24, 128), name="layer_T24"),
        # one sequence decoding through all 40 layers of a 13B-sized model, a quarter restored
        dict(block(5120, 5120, 13824, 40, 1, 64, restored=0.25), name="stack_T1"),
        # a short prompt (or a hundred sequences decoding) on a 7B-sized layer, groups of 64
        dict(block(4096, 4096, 11008, 1, 100, 64, G=64, act="bf16"), name="layer_T100_bf16_g64"),
        # an ordinary prompt on an 8B-sized layer
        dict(block(4096, 1024, 14336, 1, 512, 128), name="layer_T512"),
        # four layers of the 13B-sized model on a prompt of ragged length, a quarter restored
        dict(block(5120, 5120, 13824, 4, 1000, 64, restored=0.25), name="layers_T1000"),
        # a long prompt in bfloat16 on the 7B-sized gate/up group
        dict(group(4096, [11008] * 2, 2048, 64, act="bf16"), name="gateup_T2048_bf16"),
        # the microscaling variant: one sequence decoding, and a long prompt
        dict(group(4096, [4096] * 3, 1, 64, kind="mx"), name="mx_qkv_T1"),
        dict(group(4096, [11008] * 2, 2048, 64, act="bf16", kind="mx"), name="mx_gateup_T2048_bf16"),
        # a model is made ready unit by unit: q/k/v of width 3072 with grouped heads
        dict(offline(3072, [3072, 1024, 1024], 64, 16, 2), name="offline_d3072"),
    ]


def _log(rng, lo, hi, step=1):
    """A multiple of `step` in [lo, hi], spread over its logarithm."""
    v = math.exp(rng.uniform(math.log(lo), math.log(hi)))
    return min(hi, max(lo, int(round(v / step)) * step))


def draw(rng):
    kind = rng.choice(["group", "group", "group", "block", "mx", "offline"])
    act = rng.choice(["f16", "bf16"])
    Gs = rng.choice([64, 128, 128])
    r = rng.choice([16, 32, 64, 64, 72, 128])
    if kind == "offline":
        d = _log(rng, 512, 3072, 128)
        outs = [_log(rng, 256, 2560, 8) for _ in range(rng.randint(1, 2))]
        return offline(d, outs, rng.choice([16, 32, 64]), rng.choice([8, 16]), rng.randint(1, 2), act)
    if kind == "block":
        hidden = _log(rng, 512, 5120, 128)
        kv = rng.choice([hidden, max(128, hidden // 4 // 8 * 8)])
        inter = _log(rng, 1024, 14336, 128)
        layers = rng.randint(1, 4)
        c = block(hidden, kv, inter, layers, 1, r, Gs, act, rng.choice([0.25, 0.5, 1.0]))
        c["T"] = _log(rng, 1, max(1, min(2048, int(2.0e12 / work(c)["flops"]))))
        return c
    d = _log(rng, 256, 14336, 128)
    outs = [_log(rng, 128, 14336, 8)] * rng.randint(1, 3)
    c = group(d, outs, 1, r, Gs, act, rng.choice(["act", "act", "f32"]), rng.random() < 0.75, kind)
    c["T"] = _log(rng, 1, max(1, min(2048, int(3.8e11 / work(c)["flops"]))))
    return c


def _units(case):
    """(d_in, [d_out], restored) of every unit of a forward case."""
    if case["kind"] != "block":
        return [(case["d_in"], [int(v) for v in case["d_outs"].split(",")], bool(case.get("restore", True)))]
    h, kv, i = case["hidden"], case["kv"], case["inter"]
    units = [(h, [h, kv, kv]), (h, [h]), (h, [i, i]), (i, [h])] * case["layers"]
    order = torch.randperm(len(units), generator=torch.Generator().manual_seed(5)).tolist()
    on = set(order[:max(1, round(case["restored"] * len(units)))])
    return [(d, o, k in on) for k, (d, o) in enumerate(units)]


# ---- a pass's work ----------------------------------------------------------------------
def work(case):
    by = fl = 0
    r = case["r"]
    if case["kind"] == "offline":
        d, rows, l = case["d_in"], sum(int(v) for v in case["d_outs"].split(",")), r + case["p"]
        # in: W, Omega, the channel variances; out: codes, (s, z), tile records, A, B, sigma, scores
        by = rows * d * 4 + d * l * 8 + d * 8
        by += rows * d + rows * (d // case["G"]) * 8 + (rows + d) * r * 2 + l * 8 + 16
        # the products with the stack, one projection onto a basis, the lift
        fl = 2 * rows * d * l * (2 * case["q"] + 2) + 2 * rows * l * l + 2 * d * l * l + 2 * rows * l * r
        return {"bytes": by, "flops": fl}
    T = case["T"]
    for d, outs, on in _units(case):
        rows = sum(outs)
        scales = rows * (d // 32) if case["kind"] == "mx" else rows * (d // case["G"]) * 4
        by += rows * d // 2 + scales + T * d * 2 + T * rows * (4 if case["out"] == "f32" else 2)
        fl += 2 * T * d * rows
        if on:
            by += (rows + d) * r * 2
            fl += 2 * T * r * (d + rows)
    return {"bytes": by, "flops": fl}


def tolerance(case):
    if case["kind"] == "offline":
        # float64 throughout (sums in another order: 1e-15 apart); an element of the stored
        # factors at a rounding boundary may come out one 16-bit step away
        return {"rel": 1e-5, "max": 1e-2}
    # fp32 sums over weights that may or may not carry their 16-bit rounding, R rounded to the
    # activation type, one rounding of the output: 2.9e-4 / 1.4e-3 (binary16) and 1.7e-3 / 3.9e-3
    # (bfloat16) away from float64 sums over the stored weights
    rel, top = {"f16": (1.1e-3, 6e-3), "bf16": (6.6e-3, 1.6e-2)}[case["act"]]
    return {"rel": rel, "max": top}


# ---- inputs -----------------------------------------------------------------------------
def _words(shape, gen):
    return torch.randint(-2**31, 2**31 - 1, shape, generator=gen, device="cuda", dtype=torch.int32)


def _normal(shape, gen, std, dtype):
    return torch.randn(shape, generator=gen, device="cuda", dtype=torch.float32).mul_(std).to(dtype)


def _activations(T, d, gen, dtype):
    c = torch.exp(0.5 * torch.randn(d, generator=gen, device="cuda"))
    c[torch.randperm(d, generator=gen, device="cuda")[:d // 100]] *= 20.0
    return (torch.randn(T, d, generator=gen, device="cuda") * c).to(dtype)


def _stream():
    return torch.cuda.current_stream().cuda_stream


def _w4_codes(d_out, d, Gs, gen):
    """Packed nibbles, scales and zero-points of one module."""
    wq = _words((d_out, d // 8), gen)
    sc = torch.exp(0.1 * torch.randn(d_out, d // Gs, generator=gen, device="cuda")).mul_(STEP).to(torch.float16)
    zp = torch.randint(5, 11, (d_out, d // Gs), generator=gen, device="cuda").to(torch.float16)
    return wq, sc, zp


def _mx_codes(d_out, d, gen):
    """Packed MXFP4 elements and block scales of one module."""
    codes = _words((d_out, d // 8), gen)
    return codes, torch.randint(117, 123, (d_out, d // 32), generator=gen, device="cuda").to(torch.uint8)


def _operands(case, gen):
    """The stored operands, drawn unit by unit: (d_in, restored, X, B, iterator over (d_out, codes, A))."""
    r, dt = case["r"], ACT[case["act"]][1]

    def modules(d, d_outs, sigma):
        for d_out in d_outs:
            codes = _mx_codes(d_out, d, gen) if case["kind"] == "mx" else _w4_codes(d_out, d, case["G"], gen)
            yield d_out, codes, _normal((d_out, r), gen, math.sqrt(sigma / sum(d_outs)), dt)

    for d, d_outs, on in _units(case):
        sigma = STEP / math.sqrt(12.0) * (math.sqrt(sum(d_outs)) + math.sqrt(d))
        X, B = _activations(case["T"], d, gen, dt), _normal((r, d), gen, math.sqrt(sigma / d), dt)
        yield d, on, X, B, modules(d, d_outs, sigma)


def _prepare_forward(case, gen):
    T, r, Gs = case["T"], case["r"], case["G"]
    act = ACT[case["act"]][0]
    out, odt = ACT[case["act"] if case["out"] == "act" else case["out"]]
    keep, outs, units, mask = [], [], [], []
    shapes = _units(case)
    for n, (d, on, X, B, modules) in enumerate(_operands(case, gen)):
        if n % 4 == 0:                          # one output buffer per layer (or group), module after module
            total = sum(sum(o) for _, o, _ in shapes[n:n + 4])
            outs.append(torch.empty(T * total, dtype=odt, device="cuda"))
            used = 0
        mods = []
        for d_out, codes, A in modules:
            ptrs = [c.data_ptr() for c in codes]
            if case["kind"] == "mx":
                w = torch.empty(G.glowq_mx_prepared_bytes(d_out, d), dtype=torch.uint8, device="cuda")
                G.glowq_mx_prepare_weights(*ptrs, d_out, d, w.data_ptr(), _stream())
            else:
                w = torch.empty(G.glowq_prepared_bytes(d_out, d, Gs), dtype=torch.uint8, device="cuda")
                G.glowq_prepare_weights(*ptrs, d_out, d, Gs, w.data_ptr(), _stream())
            Y = outs[-1][used:used + T * d_out]
            mods.append(G.make_module(w.data_ptr(), A.data_ptr(), Y.data_ptr(), d_out, d_out))
            keep += [w, A]
            used += T * d_out
        units.append(G.make_unit(X.data_ptr(), B.data_ptr(), mods, T, d, r, Gs, act, out))
        mask.append(on)
        keep += [X, B]
    if case["kind"] == "mx":
        nbytes = G.glowq_mx_workspace_bytes(units[0])
    else:
        nbytes = G.glowq_workspace_bytes(units)
    ws = torch.empty(max(nbytes, 256), dtype=torch.uint8, device="cuda")
    if case["kind"] != "mx":
        G.glowq_workspace_init(ws.data_ptr(), ws.numel() // 4 * 4, _stream())
    return {"kind": case["kind"], "unit": units[0], "units": G.pack_units(units), "on": mask[0],
            "mask": G.pack_mask(mask), "ws": ws, "bytes": nbytes, "outs": outs, "keep": keep}


def _offline_inputs(case, gen):
    """fp32 weights, variances of anisotropic calibration inputs, the Gaussian test matrix."""
    d = case["d_in"]
    W = [_normal((int(v), d), gen, 0.02, torch.float32) for v in case["d_outs"].split(",")]
    variance = torch.exp(torch.randn(d, generator=gen, device="cuda", dtype=torch.float64))
    return W, variance, torch.randn(d, case["r"] + case["p"], generator=gen, device="cuda", dtype=torch.float64)


def _prepare_offline(case, gen):
    d, r, p, Gs = case["d_in"], case["r"], case["p"], case["G"]
    act, dt = ACT[case["act"]]
    mods, A, quant, prepared = [], [], [], []
    W, variance, omega = _offline_inputs(case, gen)
    for w in W:
        d_out = w.shape[0]
        A.append(torch.empty(d_out, r, dtype=dt, device="cuda"))
        quant.append((torch.empty(d_out, d // 8, dtype=torch.int32, device="cuda"),
                      torch.empty(d_out, d // Gs, dtype=torch.float16, device="cuda"),
                      torch.empty(d_out, d // Gs, dtype=torch.float16, device="cuda")))
        prepared.append(torch.empty(G.glowq_prepared_bytes(d_out, d, Gs), dtype=torch.uint8, device="cuda"))
        mods.append(G.make_module(prepared[-1].data_ptr(), A[-1].data_ptr(), 0, d_out, d_out))
    B = torch.empty(r, d, dtype=dt, device="cuda")
    unit = G.make_unit(0, B.data_ptr(), mods, 1, d, r, Gs, act, act)
    ws = torch.empty(G.glowq_factorize_workspace_bytes(unit, r, p), dtype=torch.uint8, device="cuda")
    return {"kind": "offline", "unit": unit, "d": d, "r": r, "p": p, "q": case["q"], "G": Gs, "W": W, "A": A, "B": B,
            "quant": quant, "prepared": prepared, "variance": variance, "omega": omega, "ws": ws,
            "W_ptrs": G.pack_pointers([w.data_ptr() for w in W]),
            "A_ptrs": G.pack_pointers([a.data_ptr() for a in A]),
            "scratch": torch.empty(G.GLOWQ_IMPORTANCE_SCRATCH_BYTES, dtype=torch.uint8, device="cuda"),
            "sigma": torch.empty(r + p, dtype=torch.float64, device="cuda"),
            "scores": torch.empty(2, dtype=torch.float64, device="cuda")}


def _generator(seed):
    gen = torch.Generator(device="cuda")
    gen.manual_seed(int(seed))
    return gen


def prepare(case, seed):
    gen = _generator(seed)
    return _prepare_offline(case, gen) if case["kind"] == "offline" else _prepare_forward(case, gen)


# ---- one pass ---------------------------------------------------------------------------
def run(state):
    st = _stream()
    kind = state["kind"]
    if kind == "group":
        G.glowq_group_forward(state["unit"], state["on"], state["ws"].data_ptr(), state["bytes"], st)
        return state["outs"]
    if kind == "block":
        G.glowq_block_forward(state["units"], state["mask"], state["ws"].data_ptr(), state["bytes"], st)
        return state["outs"]
    if kind == "mx":
        G.glowq_mx_group_forward(state["unit"], state["on"], state["ws"].data_ptr(), state["bytes"], st)
        return state["outs"]
    return _run_offline(state, st)


def _run_offline(s, st):
    for W, (wq, sc, zp), buf in zip(s["W"], s["quant"], s["prepared"]):
        G.glowq_quantize_rtn(W.data_ptr(), W.shape[0], s["d"], s["G"], wq.data_ptr(), sc.data_ptr(), zp.data_ptr(), st)
        G.glowq_prepare_weights(wq.data_ptr(), sc.data_ptr(), zp.data_ptr(), W.shape[0], s["d"], s["G"],
                                buf.data_ptr(), st)
    G.glowq_factorize_unit(s["unit"], s["W_ptrs"], s["variance"].data_ptr(), s["r"], s["p"], s["q"],
                           s["omega"].data_ptr(), s["ws"].data_ptr(), s["ws"].numel(), s["A_ptrs"],
                           s["B"].data_ptr(), s["sigma"].data_ptr(), st)
    G.glowq_unit_importance(s["unit"], s["W_ptrs"], s["scratch"].data_ptr(), s["scores"].data_ptr(), st)
    # a rank's pair (A[:, j], B[j, :]) is defined up to a common sign: stored with the first
    # element of B's row positive, so that two models can be compared
    sign = torch.where(s["B"][:, :1] < 0, -1, 1).to(s["B"].dtype)
    B = s["B"] * sign
    A = [a * sign.T for a in s["A"]]
    return {"codes": [q[0] for q in s["quant"]], "scales": [q[1] for q in s["quant"]],
            "zeros": [q[2] for q in s["quant"]], "prepared": s["prepared"], "A": A, "B": B,
            "sigma": s["sigma"], "scores": s["scores"]}


# ---- the same in 64 bits ----------------------------------------------------------------
def exact(case, seed):
    gen = _generator(seed)
    return _exact_offline(case, gen) if case["kind"] == "offline" else _exact_forward(case, gen)


def _nibbles(words):
    """[rows][d / 8] words -> [rows][d] codes, element 8 j + e in bits 4 e .. 4 e + 3 of word j."""
    shift = torch.arange(0, 32, 4, device=words.device, dtype=torch.int32)
    return ((words.unsqueeze(-1) >> shift) & 15).reshape(words.shape[0], -1)


def _mx_activations(X):
    """MXFP8 values of X (the format's own rounding is part of the result, not an error of it)."""
    v = X.double().reshape(X.shape[0], -1, 32)
    top = v.abs().amax(dim=2, keepdim=True)
    power = torch.where(top > 0, torch.floor(torch.log2(top)) - 8.0, torch.zeros_like(top)).clamp(-127, 127)
    q = torch.ldexp(v, -power).clamp(-448, 448).to(torch.float32).to(torch.float8_e4m3fn).double()
    return torch.ldexp(q, power).reshape(X.shape)


def _weight(case, codes):
    """The stored weight: (q - z) s in the activation type, or element times block scale."""
    q = _nibbles(codes[0])
    if case["kind"] == "mx":
        values = torch.tensor([0, .5, 1, 1.5, 2, 3, 4, 6], dtype=torch.float64, device="cuda")
        values = torch.cat([values, -values])
        return values[q.long()] * torch.exp2(codes[1].double() - 127.0).repeat_interleave(32, dim=1)
    s, z = (c.double().repeat_interleave(case["G"], dim=1) for c in codes[1:])
    return ((q - z) * s).to(ACT[case["act"]][1]).double()


def _exact_forward(case, gen):
    outs = []
    for n, (d, on, X, B, modules) in enumerate(_operands(case, gen)):
        if n % 4 == 0:
            outs.append([])
        x = X.double()
        R = x @ B.double().T
        if case["kind"] == "mx":
            x = _mx_activations(X)
        for _, codes, A in modules:
            y = x @ _weight(case, codes).T
            outs[-1].append((y + R @ A.double().T if on else y).reshape(-1))
    return [torch.cat(o) for o in outs]


def _exact_offline(case, gen):
    """RTN, Alg. 1 without re-orthonormalisation between the power steps, scores of the stored factors."""
    W, variance, omega = _offline_inputs(case, gen)
    r, Gs, dt = case["r"], case["G"], ACT[case["act"]][1]
    scales, zeros, errors = [], [], []
    for w in W:
        v = w.double().reshape(w.shape[0], -1, Gs)
        lo, hi = v.amin(dim=2).clamp(max=0.0), v.amax(dim=2).clamp(min=0.0)
        s = ((hi - lo) / 15.0).clamp(min=2.0**-14).to(torch.float16)
        z = torch.round(-lo / s.double()).clamp(0, 15)
        q = (torch.round(v / s.double().unsqueeze(2)) + z.unsqueeze(2)).clamp(0, 15)
        stored = ((q - z.unsqueeze(2)) * s.double().unsqueeze(2)).to(dt).double()
        scales.append(s.double())
        zeros.append(z)
        errors.append((v - stored).reshape(w.shape))
    E = torch.cat(errors)
    M = E * variance.sqrt()
    Y = M @ omega
    for _ in range(case["q"]):
        Y = M @ (M.T @ Y)
    Q = torch.linalg.qr(Y.cpu()).Q.to(Y.device)
    U, S, Vt = (t.cuda() for t in torch.linalg.svd((Q.T @ M).cpu(), full_matrices=False))
    root = S[:r].sqrt()
    A, B = Q @ (U[:, :r] * root), root[:, None] * Vt[:r] / variance.sqrt()
    sign = torch.where(B[:, :1] < 0, -1.0, 1.0).double()
    A, B = A * sign.T, B * sign
    captured = (A.to(dt).double().square().sum(0) * B.to(dt).double().square().sum(1)).sum()
    energy = E.square().sum()
    whole = sum(w.double().square().sum() for w in W)
    none = [None] * len(W)
    return {"codes": none, "scales": scales, "zeros": zeros, "prepared": none,
            "A": list(A.split([w.shape[0] for w in W])), "B": B, "sigma": S,
            "scores": torch.stack([energy / whole, captured / energy])}
