"""The workloads whose speed this package is judged by, one pass of each through
the public entry points, with inputs, required work, tolerances and results in
64 bits.

A case is a dict: ``kind`` (the entry point and how a program calls it), the
format (``M`` codebooks of ``2^B`` codewords of ``g`` values, ``packed`` codes
or not) and the sizes.  The kinds and what each stands for:

gemv     one layer's matrix-vector product, called eagerly: the smallest call a
         program makes (a single linear layer at batch 1), where the launch and
         the fixed cost of a kernel count as much as the bytes.  2x8 over
         row-major codes, bit-packed 12-bit codes (the 3-bit models) and groups
         of 16 (the codebooks-versus-groups ablation).
decode   the linear layers of several transformer blocks at batch 1 (q/k/v
         grouped, o, gate/up grouped, down), codes stored tiled (8-bit) or
         chunk-sorted (one large codebook) once at load time, the launches
         captured once in a graph and replayed per token.  Enough blocks that
         the codes come from HBM, as they do in a whole model.
batch    one layer for a few activation rows: several sequences decoded
         together, or a short draft being verified.
prefill  one layer for a prompt, with the caller's workspace kept between calls
         (the weights are rebuilt in every call).
backward codebook and scale gradients of one layer for a fine-tuning
         micro-batch.
beam     Phase 1 of the quantizer: one sweep of the beam search over a layer.
"""
from __future__ import annotations

import math

import torch

import paper_2401_06118_amd as aqlm
from paper_2401_06118_amd import synth

DEV = "cuda"


def listed():
    return [
        # one 4096 x 4096 attention projection of a 7B model at batch 1
        dict(name="gemv_2x8_4096", kind="gemv", M=2, B=8, g=8, packed=False, d_out=4096, d_in=4096),
        # a 7B gate projection stored at 3 bits per weight, codes bit-packed
        dict(name="gemv_2x12_packed_gate", kind="gemv", M=2, B=12, g=8, packed=True, d_out=11008, d_in=4096),
        # the larger-group setting of the ablation (2 bits from four codebooks)
        dict(name="gemv_4x8_g16_gate", kind="gemv", M=4, B=8, g=16, packed=False, d_out=11008, d_in=4096),
        # token generation, 7B and 70B shapes, 2 bits: the headline workload
        dict(name="decode_7b_2x8", kind="decode", M=2, B=8, hidden=4096, kv=4096, ffn=11008, blocks=8),
        dict(name="decode_70b_2x8", kind="decode", M=2, B=8, hidden=8192, kv=1024, ffn=28672, blocks=3),
        # token generation with the most accurate 2-bit setting
        dict(name="decode_7b_1x16", kind="decode", M=1, B=16, hidden=4096, kv=4096, ffn=11008, blocks=3),
        # sixteen sequences at once, 4-bit codes (tiled), gate projection
        dict(name="batch16_4x8_gate", kind="batch", M=4, B=8, n=16, d_out=11008, d_in=4096),
        # a handful of rows against the 1x16 down projection
        dict(name="batch5_1x16_down", kind="batch", M=1, B=16, n=5, d_out=4096, d_in=11008),
        # a full prompt and a short ragged one
        dict(name="prefill2048_2x8_gate", kind="prefill", M=2, B=8, n=2048, d_out=11008, d_in=4096),
        dict(name="prefill333_1x16_down", kind="prefill", M=1, B=16, n=333, d_out=4096, d_in=11008),
        # a fine-tuning micro-batch
        dict(name="backward2048_2x8_gate", kind="backward", M=2, B=8, n=2048, d_out=11008, d_in=4096),
        # one sweep of Phase 1
        dict(name="beam4_2x8_4096x1024", kind="beam", M=2, B=8, d_out=4096, d_in=1024, beam=4),
    ]


def _log(rng, lo, hi, step=1):
    """A multiple of ``step`` in [lo, hi], spread over the logarithm."""
    v = math.exp(rng.uniform(math.log(lo), math.log(hi + step)))
    return max(lo, min(hi, int(v) // step * step))


def draw(rng):
    kind = rng.choice(["gemv", "decode", "batch", "prefill", "backward", "beam"])
    if kind == "gemv":
        M, B, g, packed = rng.choice([(2, 8, 8, False), (4, 8, 8, False), (2, 12, 8, True), (1, 16, 8, False),
                                      (4, 8, 16, False), (8, 8, 32, False)])
        return dict(kind=kind, M=M, B=B, g=g, packed=packed, d_out=_log(rng, 1000, 14336),
                    d_in=_log(rng, 1024, 11264, g))
    if kind == "decode":
        M, B = rng.choice([(2, 8), (2, 8), (1, 16)])
        hidden = _log(rng, 2048, 8192 if B == 8 else 4096, 128)
        ffn = int(hidden * rng.uniform(2.6, 3.5)) // 128 * 128
        kv = rng.choice([hidden, hidden // 4 // 64 * 64, hidden // 8 // 64 * 64])
        per_block = (2 * hidden * hidden + 2 * kv * hidden + 3 * hidden * ffn) // 8 * M * (2 if B > 8 else 1)
        return dict(kind=kind, M=M, B=B, hidden=hidden, kv=kv, ffn=ffn,
                    blocks=max(1, min(10, (450 << 20 if B == 8 else 150 << 20) // per_block)))
    if kind == "batch":
        M, B = rng.choice([(2, 8), (4, 8), (1, 16), (2, 12)])
        return dict(kind=kind, M=M, B=B, n=_log(rng, 2, 48), d_out=_log(rng, 1000, 14336),
                    d_in=_log(rng, 1024, 11264, 8))
    if kind == "prefill":
        M, B = rng.choice([(2, 8), (4, 8), (1, 16), (2, 12)])
        d_out, d_in = _log(rng, 1024, 14336), _log(rng, 1024, 11264, 64)
        return dict(kind=kind, M=M, B=B, n=_log(rng, 64, max(64, min(4096, 2048 * 11008 * 4096 // (d_out * d_in)))),
                    d_out=d_out, d_in=d_in)
    if kind == "backward":
        M = rng.choice([1, 2, 4])
        d_out, d_in = _log(rng, 1024, 11008, 8), _log(rng, 1024, 11008, 8)
        n = _log(rng, 64, max(64, min(4096, 2048 * 11008 * 4096 // (d_out * d_in))))
        return dict(kind=kind, M=M, B=8, n=n, d_out=d_out, d_in=d_in)
    M, beam = rng.choice([1, 2, 4]), rng.choice([1, 2, 4, 4, 8])
    d_in = _log(rng, 256, 1536, 8)
    d_out = _log(rng, 128, max(128, min(4096, 4096 * 1024 * 1024 * 2 * 4 // (d_in * d_in * M * beam))))
    return dict(kind=kind, M=M, B=8, d_out=d_out, d_in=d_in, beam=beam)


def _grouped(case):
    """(d_out, d_in) of a block's layers, grouped as they are launched."""
    h, kv, f = case["hidden"], case["kv"], case["ffn"]
    return [[(h, h), (kv, h), (kv, h)], [(h, h)], [(f, h), (f, h)], [(h, f)]]


def _seed(seed, k):
    return (seed * 1000003 + k * 7919 + 17) % (1 << 62)


def _block_inputs(case, seed):
    """The layers of all blocks, launch after launch: each launch's layers read
    one activation, as in a model."""
    k = 0
    for _ in range(case["blocks"]):
        for launch in _grouped(case):
            x, out = None, []
            for d_out, d_in in launch:
                codes, cb, sc, xk = synth.device_layer(_seed(seed, k), d_out, d_in, case["M"], case["B"], device=DEV)
                x = xk[0] if x is None else x
                out.append((codes, cb, sc, x))
                k += 1
            yield out


def _layer(case, seed, n):
    M, B, g = case["M"], case["B"], case.get("g", 8)
    make = synth.device_packed_layer if case.get("packed") else synth.device_layer
    return make(_seed(seed, 0), case["d_out"], case["d_in"], M, B, g, n, device=DEV)


def _beam_inputs(case, seed):
    """A layer whose weights lie near a reconstruction of the given codebooks
    (Phase 1 starts from initialised codes: here the true ones with a quarter
    redrawn), and H from 512 calibration vectors."""
    d_out, d_in, M = case["d_out"], case["d_in"], case["M"]
    codes, cb, sc, _ = synth.device_layer(_seed(seed, 0), d_out, d_in, M, 8, device=DEV)
    gen = torch.Generator(device=DEV)
    gen.manual_seed(_seed(seed, 1))
    w = torch.zeros((d_out, d_in // 8, 8), device=DEV)
    for m in range(M):
        w += cb[m].float()[codes[:, :, m].long()]
    w = w.reshape(d_out, d_in) * sc.float()[:, None]
    w = w + 0.01 * torch.randn(w.shape, device=DEV, generator=gen)
    x = torch.randn((d_in, 512), device=DEV, generator=gen)
    # integer-valued calibration keeps H exact in fp32
    x = (x * 8).round().clamp(-32, 32)
    h = (x.double() @ x.double().T).float() / 64
    other = torch.randint(0, 256, codes.shape, dtype=torch.uint8, device=DEV, generator=gen)
    redraw = torch.rand(codes.shape, device=DEV, generator=gen) < 0.25
    codes = torch.where(redraw, other, codes).contiguous()
    return w.contiguous(), h.contiguous(), codes, cb, sc


def prepare(case, seed):
    kind = case["kind"]
    if kind == "gemv":
        codes, cb, sc, x = _layer(case, seed, 1)
        return dict(kind=kind, args=(codes, cb, sc, x[0]))
    if kind == "decode":
        launches, ys = [], []
        tiled = case["B"] == 8
        for layers in _block_inputs(case, seed):
            probs = []
            for codes, cb, sc, x in layers:
                y = torch.empty(codes.shape[0], dtype=torch.float16, device=DEV)
                stored = aqlm.TiledCodes(codes, cb, sc) if tiled else aqlm.SortedCodes(codes, cb, sc)
                probs.append((stored, x, y))
                ys.append(y)
            launches.append(probs)
        step = aqlm.gemv_tiled_grouped if tiled else aqlm.gemv_sorted_grouped
        kw = {}
        if not tiled:
            # the workspace this graph owns, sized for its largest launch
            need = max(int(aqlm._lib.load().aqlm_gemv_sorted_workspace_bytes(
                sum(s.d_out for s, _, _ in p), case["M"], case["B"])) for p in launches)
            kw["workspace"] = torch.zeros(need, dtype=torch.uint8, device=DEV)
        side = torch.cuda.Stream()
        side.wait_stream(torch.cuda.current_stream())
        with torch.cuda.stream(side):
            for probs in launches:
                step(probs, **kw)
        torch.cuda.current_stream().wait_stream(side)
        torch.cuda.synchronize()
        graph = torch.cuda.CUDAGraph()
        with torch.cuda.graph(graph):
            for probs in launches:
                step(probs, **kw)
        return dict(kind=kind, graph=graph, ys=ys, keep=(launches, kw))
    if kind == "batch":
        codes, cb, sc, x = _layer(case, seed, case["n"])
        if case["B"] == 8:
            return dict(kind=kind, tiled=aqlm.TiledCodes(codes, cb, sc), x=x)
        return dict(kind=kind, args=(codes, cb, sc, x))
    if kind == "prefill":
        codes, cb, sc, x = _layer(case, seed, case["n"])
        need = aqlm.gemm_workspace_bytes(codes, cb, sc, case["n"])
        ws = torch.empty(max(need, 16), dtype=torch.uint8, device=DEV)
        return dict(kind=kind, args=(codes, cb, sc, x), ws=ws)
    if kind == "backward":
        codes, cb, sc, x = _layer(case, seed, case["n"])
        gen = torch.Generator(device=DEV)
        gen.manual_seed(_seed(seed, 2))
        dy = torch.randn((case["n"], case["d_out"]), device=DEV, generator=gen).to(torch.float16)
        return dict(kind=kind, args=(codes, cb, sc, x, dy))
    w, h, codes, cb, sc = _beam_inputs(case, seed)
    return dict(kind=kind, w=w, h=h, codes=codes, cb=cb, sc=sc, beam=case["beam"])


def run(state):
    kind = state["kind"]
    if kind == "gemv":
        return aqlm.gemv(*state["args"])
    if kind == "decode":
        state["graph"].replay()
        return state["ys"]
    if kind == "batch":
        if "tiled" in state:
            return state["tiled"].gemm_small_batch(state["x"])
        return aqlm.gemm_small_batch(*state["args"])
    if kind == "prefill":
        return aqlm.gemm(*state["args"], workspace=state["ws"])
    if kind == "backward":
        dcb, ds = aqlm.backward(*state["args"])
        return [dcb, ds]
    codes = state["codes"].clone()  # (searched in place)
    loss = aqlm.beam_search(state["w"], state["h"], codes, state["cb"], state["sc"], beam=state["beam"])
    return [codes, loss]


def _row_bytes(d_in, M, B, g, packed):
    n = d_in // g * M
    if packed:
        return (n * B + 31) // 32 * 4
    return n * (2 if B > 8 else 1)


def _layer_bytes(d_out, d_in, M, B, g=8, packed=False, n=1):
    return (d_out * _row_bytes(d_in, M, B, g, packed) + M * (1 << B) * g * 2 + 2 * d_out + 2 * n * d_in
            + 2 * n * d_out)


def work(case):
    kind, M, B = case["kind"], case["M"], case["B"]
    if kind == "decode":
        b = f = 0
        for launch in _grouped(case):
            for d_out, d_in in launch:
                b += _layer_bytes(d_out, d_in, M, B)
                f += 2 * d_out * d_in
        return {"bytes": b * case["blocks"], "flops": f * case["blocks"]}
    d_out, d_in = case["d_out"], case["d_in"]
    if kind == "beam":
        # one 8-wide inner product per candidate, one rank-8 update of H r per
        # kept configuration, the first and last loss of each row
        steps = d_in // 8 * M
        per_row = steps * case["beam"] * (256 * 16 + 16 * d_in) + 4 * d_in * d_in
        return {"bytes": d_out * d_in * 4 + d_in * d_in * 4 + 2 * d_out * steps + M * 4096 + 6 * d_out,
                "flops": d_out * per_row}
    n = case.get("n", 1)
    byt = _layer_bytes(d_out, d_in, M, B, case.get("g", 8), case.get("packed", False), n)
    if kind == "backward":
        byt += M * 256 * 8 * 4 + 4 * d_out
    return {"bytes": byt, "flops": 2 * n * d_out * d_in}


def tolerance(case):
    if case["kind"] == "backward":
        # fp32 sums in any order: 4.7e-7 against 64 bits, 3.5e-7 (max 1.6e-6)
        # between two runs of one build
        return {"rel": 2e-6, "max": 1e-5}
    if case["kind"] == "beam":
        # Scores that differ by less than fp32 resolves may be ranked either
        # way, and a row's path then parts for good.  Against the search in 64
        # bits over nine shapes x two seeds: up to 0.0018 of the codes (0.6 %
        # of the rows), loss rel 9.9e-3, max 0.19.
        return {"rel": 4e-2, "max": 0.8, "differ": 0.008}
    # fp16 results of fp32 sums: 2.1e-4 against 64 bits (the final rounding)
    return {"rel": 8.5e-4, "max": 2e-3}


def _unpack(words, d_in, M, B):
    """Codes of bit-packed rows (code k of a row at bits [k B, k B + B))."""
    n = d_in // 8 * M
    bit = torch.arange(n, device=DEV) * B
    w = words.long() & 0xFFFFFFFF
    lo, sh = bit // 32, bit % 32
    hi = (lo + 1).clamp(max=words.shape[1] - 1)
    both = w[:, lo] | (w[:, hi] << 32)
    return ((both >> sh) & ((1 << B) - 1)).reshape(words.shape[0], -1, M)


def _weights(codes, cb, d_in, rows):
    """fp64 codeword sums [rows, d_in] of the given row range (no scales)."""
    M, entries, _ = cb.shape
    c = codes[rows]
    if c.dim() == 2:
        c = _unpack(c, d_in, M, entries.bit_length() - 1)
    c = c.long() & (entries - 1)
    u = cb[0].double()[c[:, :, 0]]
    for m in range(1, M):
        u = u + cb[m].double()[c[:, :, m]]
    return u.reshape(c.shape[0], d_in)


def _product(codes, cb, sc, x, rounded):
    """X W^T in fp64, W from Eq. 2 (``rounded``: to fp16 first, as the
    workspace product defines it)."""
    d_out, d_in = codes.shape[0], x.shape[-1]
    xd = x.double().reshape(-1, d_in)
    out = torch.empty((xd.shape[0], d_out), dtype=torch.float64, device=DEV)
    for r0 in range(0, d_out, 2048):
        rows = slice(r0, min(r0 + 2048, d_out))
        w = _weights(codes, cb, d_in, rows) * sc[rows].double()[:, None]
        if rounded:
            w = w.half().double()
        out[:, rows] = xd @ w.T
    return out.reshape(*x.shape[:-1], d_out)


def _exact_backward(codes, cb, sc, x, dy):
    d_out, d_in = codes.shape[0], x.shape[1]
    M = cb.shape[0]
    dcb = torch.zeros(cb.shape, dtype=torch.float64, device=DEV)
    ds = torch.empty(d_out, dtype=torch.float64, device=DEV)
    xd = x.double()
    for r0 in range(0, d_out, 1024):
        rows = slice(r0, min(r0 + 1024, d_out))
        G = dy[:, rows].double().T.contiguous() @ xd
        u = _weights(codes, cb, d_in, rows)
        ds[rows] = (G * u).sum(1)
        sg = (G * sc[rows].double()[:, None]).reshape(-1, 8)
        for m in range(M):
            idx = codes[rows, :, m].reshape(-1).long()
            order = torch.argsort(idx)
            total = torch.cat([torch.zeros((1, 8), dtype=torch.float64, device=DEV), sg[order].cumsum(0)])
            ends = torch.searchsorted(idx[order], torch.arange(257, device=DEV))
            dcb[m] += total[ends[1:]] - total[ends[:-1]]
    return [dcb, ds]


def _exact_beam(w, h, codes, cb, sc, beam):
    """The search in fp64, all rows at once: every position in order, every
    codeword for every configuration, the ``beam`` best distinct ones kept
    (ties: earlier configuration, then smaller code)."""
    R, G, M = codes.shape
    w, h, s = w.double(), h.double(), sc.double()
    cbd = cb.double()
    conf = codes.long()[:, None].clone()                                    # [R, nb, G, M]

    def residual(c):
        u = sum(cbd[m][c[..., m]] for m in range(M))                         # [..., G, 8]
        return w.reshape(R, *([1] * (c.dim() - 3)), G, 8) - s.reshape(R, *([1] * (c.dim() - 1))) * u

    hr = (residual(conf).reshape(-1, G * 8) @ h).reshape(R, 1, -1)
    loss = (residual(conf).reshape(R, 1, -1) * hr).sum(-1)                   # [R, nb]
    ar = torch.arange(R, device=DEV)[:, None]
    for j in range(G):
        sl = slice(8 * j, 8 * j + 8)
        hjj = h[sl, sl]
        for m in range(M):
            nb = conf.shape[1]
            old = conf[:, :, j, m]
            d = s[:, None, None, None] * (cbd[m][None, None] - cbd[m][old][:, :, None])   # [R, nb, 256, 8]
            dl = ((d.reshape(-1, 8) @ hjj).reshape(d.shape) * d).sum(-1) \
                - 2 * torch.bmm(d.reshape(R * nb, 256, 8), hr[:, :, sl].reshape(R * nb, 8, 1)).reshape(R, nb, 256)
            score = loss[:, :, None] + dl
            rest = conf.clone()
            rest[:, :, j, m] = 0
            rest = rest.reshape(R, nb, -1)
            for b in range(1, nb):  # equal elsewhere to an earlier configuration: its candidates stand
                same = (rest[:, b:b + 1] == rest[:, :b]).all(-1).any(1)
                score[:, b] = torch.where(same[:, None], torch.inf, score[:, b])
            val, idx = torch.sort(score.reshape(R, -1), dim=1, stable=True)
            keep = min(beam, nb * 256)
            val, idx = val[:, :keep], idx[:, :keep]
            par, code = idx // 256, idx % 256
            step = d[ar, par, code]                                           # [R, keep, 8]
            conf = conf[ar, par].clone()
            conf[:, :, j, m] = code
            hr = hr[ar, par] - (step.reshape(-1, 8) @ h[sl]).reshape(R, keep, -1)
            loss = val
    best = conf[:, 0]
    r = residual(best).reshape(R, -1)
    return best, ((r @ h) * r).sum(-1)


def exact(case, seed):
    kind = case["kind"]
    if kind == "gemv":
        codes, cb, sc, x = _layer(case, seed, 1)
        if case["g"] != 8:
            g, k = case["g"], case["g"] // 8
            # a codeword of g values is k chunks of 8, a code serves k groups
            out = torch.empty(case["d_out"], dtype=torch.float64, device=DEV)
            u = sum(cb[m].double()[codes[:, :, m].long()] for m in range(case["M"])).reshape(case["d_out"], -1)
            out[:] = (u @ x[0].double()) * sc.double()
            return out
        return _product(codes, cb, sc, x[0], False)
    if kind == "decode":
        ys = []
        for layers in _block_inputs(case, seed):
            for codes, cb, sc, x in layers:
                ys.append(_product(codes, cb, sc, x, False))
        return ys
    if kind in ("batch", "prefill"):
        codes, cb, sc, x = _layer(case, seed, case["n"])
        return _product(codes, cb, sc, x, kind == "prefill")
    if kind == "backward":
        codes, cb, sc, x = _layer(case, seed, case["n"])
        gen = torch.Generator(device=DEV)
        gen.manual_seed(_seed(seed, 2))
        dy = torch.randn((case["n"], case["d_out"]), device=DEV, generator=gen).to(torch.float16)
        return _exact_backward(codes, cb, sc, x, dy)
    w, h, codes, cb, sc = _beam_inputs(case, seed)
    # (codes are whole numbers: near-ties may go either way; the loss is that
    # of the search in fp64)
    return [None, _exact_beam(w, h, codes, cb, sc, case["beam"])[1]]
